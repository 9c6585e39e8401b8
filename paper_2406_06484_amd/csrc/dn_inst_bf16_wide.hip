// bf16 instantiation for d_k = d_v = 256: scans with 16 to 64 state columns per workgroup, the backward's chunk
// kernel with blocks of 32; plain, gated and fused-prologue variants
#include "dn_launch.hpp"
namespace dn {
DN_INSTANTIATE(bf16, 256, 256)
} // namespace dn
