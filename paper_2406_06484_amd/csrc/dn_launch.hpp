// Launch sequences of the forward and backward pass for one (T, DK, DV); included only by the
// instantiation files.
#pragma once
#include <atomic>
#include <tuple>

#include "dn_host.hpp"
#include "dn_kernels.hpp"
#include "dn_chunk_bf16.hpp"
#include "dn_chunk_local.hpp"

namespace dn {

constexpr size_t kLdsPerWorkgroup = 160 * 1024; // gfx950

// Raises the dynamic-LDS limit of `kernel` once per device and call site (every call site names one kernel
// instantiation), then launches it; returns the launch's own status, so an error some earlier, unrelated call left
// behind is neither reported as this launch's nor cleared.
template <typename... Params, typename... Args>
static inline int launch_kernel(void (*kernel)(Params...), std::atomic<uint64_t> &lds_set, int device, dim3 grid, int nthreads,
                                size_t lds, hipStream_t stream, Args... args) {
    const uint64_t bit = 1ull << (device & 63);
    if (lds > 0 && !(lds_set.load(std::memory_order_relaxed) & bit)) { // (a call site always asks for the same amount)
        const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e != hipSuccess) return (int)e;
        lds_set.fetch_or(bit, std::memory_order_relaxed);
    }
    std::tuple<Params...> held(static_cast<Params>(args)...); // the kernel's own parameter types, by value
    void *ptrs[sizeof...(Params)];
    int i = 0;
    std::apply([&](auto &...a) { ((ptrs[i++] = (void *)&a), ...); }, held);
    return (int)hipLaunchKernel(reinterpret_cast<const void *>(kernel), grid, dim3(nthreads), ptrs, lds, stream);
}

#define DN_LAUNCH(kernel, grid, lds, ...) DN_LAUNCH_NT(kernel, grid, NTHR, lds, __VA_ARGS__)
#define DN_LAUNCH_NT(kernel, grid, nthreads, lds, ...)                                                        \
    do {                                                                                                      \
        static std::atomic<uint64_t> lds_set_{0};                                                             \
        prof_begin(#kernel, pb.stream);                                                                       \
        const int e_ = launch_kernel(kernel, lds_set_, pb.device, grid, nthreads, lds, pb.stream, __VA_ARGS__); \
        prof_end(pb.stream);                                                                                  \
        if (e_) return e_;                                                                                    \
    } while (0)

static inline SeqMap make_map(const Problem &pb) {
    SeqMap sm;
    sm.cu = pb.cu; sm.coff = pb.coff; sm.N = pb.N; sm.L = pb.L; sm.ncd = (pb.L + C - 1) / C;
    sm.order = pb.cu ? pb.coff + pb.N + 1 : nullptr;
    // (pb.cu is the bounded copy of the caller's offsets that k_chunk_offsets leaves behind the order)
    return sm;
}

static inline int launch_offsets(const Problem &pb) {
    if (!pb.cu) return 0;
    DN_LAUNCH(k_chunk_offsets, dim3(1), 0, pb.cu_user, pb.N, pb.L, pb.coff);
    return 0;
}

// chain waves of the widest scan workgroup: 64 state columns
template <typename T, int DV> constexpr int kMostChainWaves = sizeof(T) == 4 ? 2 : DV < 64 ? DV / 16 : 4; // (fp32: 32 columns)

// Which chunk kernel: in bf16 up to d_k = 128 the one whose tiles travel straight to the LDS (both sides' times at every head size: dn_chunk_bf16.hpp); fp32, and d_k = 256, where the masked rows'
// extra work per block of 32 state columns costs that kernel more than it gains (16 384 tokens of 8 heads, none / a tenth / padding masked: tiles
// through registers 215, 250, 247 us, straight to the LDS 204, 326, 305), keep the one that holds them in registers.
template <typename T, int DK> constexpr bool kDmaChunk = sizeof(T) == 2 && DK <= 128;
template <typename T, int DK, int DV> constexpr size_t local_lds() {
    if constexpr (kDmaChunk<T, DK>) return ChunkSmem<DK, DV>::bytes;
    else return cmax(LocalSmem<T, DK, DV>::bytes, LocalSmem<T, DK, DV>::bytes_pro);
}
template <typename T, int DK, int DV> constexpr size_t LocalLds = local_lds<T, DK, DV>();
template <typename T, int DK, int DV> constexpr int local_wpc() {
    if constexpr (kDmaChunk<T, DK>) return ChunkSmem<DK, DV>::WPC;
    else return 1;
}
template <typename T, int DK, int DV, int VAR>
__global__ __launch_bounds__(NTC) __attribute__((amdgpu_waves_per_eu(2 * local_wpc<T, DK, DV>(), 2 * local_wpc<T, DK, DV>()))) void k_bwd_local(SeqMap sm, int H, Ptrs p, int chunks_total) {
    if constexpr (kDmaChunk<T, DK>) bwd_local_bf16<DK, DV, VAR>(sm, H, p, chunks_total);
    else bwd_local_regs<T, DK, DV, VAR>(sm, H, p, chunks_total);
}

template <typename T, int DK, int DV> size_t max_lds_bytes() {
    constexpr size_t scan = ScanSmem<T, DK, kMostChainWaves<T, DV>>::bytes;
    static_assert(PrepSmem<T, DK, DV>::bytes <= kLdsPerWorkgroup, "k_wy_prep LDS");
    static_assert(scan <= kLdsPerWorkgroup, "scan LDS");
    size_t m = PrepSmem<T, DK, DV>::bytes;
    if (scan > m) m = scan;
    static_assert(LocalLds<T, DK, DV> <= kLdsPerWorkgroup, "k_bwd_local LDS");
    if (LocalLds<T, DK, DV> > m) m = LocalLds<T, DK, DV>;
    return m;
}

// A scan over `passes` grids of nchains chains takes the fewest chain waves per workgroup (columns over 16) with which the
// workgroups still fit the chip at once: the fewer share a CU's LDS, the shorter a step.  With the fewest and with the most waves, scan
// alone, in us: bf16, 16 heads of 128, 1 x 1000 tokens 21.7 and 29.8, 2 x 500 forward 15.4 and 19.1, reverse 16.2 and 20.3; 8 heads,
// 1 x 300 10.1 and 13.3; fp32, 1 x 256 of 2 heads of 64, 21.3 and 24.0.  Past one round of the chip the widest is taken: q and k
// are then read by the fewest workgroups, and a CU holds one workgroup of any width.  With 64, 32 and 16 columns, at 32 x 512 tokens of width 2048: d = 64,
// forward 64 101 184, reverse 81 120 207; d = 128 72 116 199 and 99 151 257; at 32 x 128: d = 64 27 37 63 and 32 43 76, d = 128 34 44 79 and 40 53 94.
template <typename T, int DV> static inline int chain_waves(const Problem &pb, long nchains, int passes) {
    for (int w = 1; w < kMostChainWaves<T, DV>; w *= 2)
        if ((long)chain_grid((int)nchains, DV / (16 * w)) * passes <= pb.num_cus) return w;
    return kMostChainWaves<T, DV>;
}
// launches the scan kernel<T, DK, DV, gated, ncw> over `passes` grids; half_ = workgroups of one pass, the last
// argument of the kernels of several passes
#define DN_LAUNCH_SCAN_W(kernel, DIR, W, passes, ...)                                                                                  \
    do {                                                                                                                          \
        const int half_ = chain_grid(sm.N * pb.H, DV / (16 * (W)));                                                               \
        if (p.g) DN_LAUNCH_NT((kernel<T, DK, DV, true, W>), dim3(half_ * (passes)), (kScanThreads<T, DK, DIR, W>), (ScanSmem<T, DK, W>::bytes), __VA_ARGS__); \
        else DN_LAUNCH_NT((kernel<T, DK, DV, false, W>), dim3(half_ * (passes)), (kScanThreads<T, DK, DIR, W>), (ScanSmem<T, DK, W>::bytes), __VA_ARGS__);    \
    } while (0)
#define DN_LAUNCH_SCAN(kernel, DIR, passes, ...)                                                \
    do {                                                                                   \
        const int ncw_ = chain_waves<T, DV>(pb, (long)sm.N * pb.H, passes);                       \
        if (ncw_ == 1) DN_LAUNCH_SCAN_W(kernel, DIR, 1, passes, __VA_ARGS__);                   \
        else if (kMostChainWaves<T, DV> == 2 || ncw_ == 2) DN_LAUNCH_SCAN_W(kernel, DIR, 2, passes, __VA_ARGS__); \
        else DN_LAUNCH_SCAN_W(kernel, DIR, (kMostChainWaves<T, DV>), passes, __VA_ARGS__);          \
    } while (0)
// what the scans see: with the prologue, the mapped q and k in the workspace (beta stays the logit)
static inline Ptrs scan_ptrs(const Ptrs &p) {
    Ptrs ps = p;
    if (p.pro) { ps.q = p.Qm; ps.k = p.Km; }
    return ps;
}

template <typename T, int DK, int DV> int launch_prep(const Problem &pb, const SeqMap &sm, const Ptrs &p) {
    const dim3 grid((unsigned)pb.chunks_ub * (unsigned)pb.H); // (rows * H < 2^31)
    if (p.pro) DN_LAUNCH((k_wy_prep<T, DK, DV, true>), grid, (PrepSmem<T, DK, DV>::bytes), sm, pb.H, p);
    else DN_LAUNCH((k_wy_prep<T, DK, DV, false>), grid, (PrepSmem<T, DK, DV>::bytes), sm, pb.H, p);
    return 0;
}

template <typename T, int DK, int DV> int run_fwd(const Problem &pb, const Ptrs &p) {
    if (pb.N == 0) return 0;
    if (pb.chunks_ub == 0) { // no tokens at all: the state passes through (section 2.2: nothing is written)
        if (p.ST) {
            const long count = (long)pb.N * pb.H * DK * DV;
            DN_LAUNCH(k_state_copy, dim3((unsigned)((count + 4 * NTHR - 1) / (4 * NTHR))), 0, p.ST, p.S0, count);
        }
        return 0;
    }
    SeqMap sm = make_map(pb);
    if (int e = launch_offsets(pb)) return e;
    if (int e = launch_prep<T, DK, DV>(pb, sm, p)) return e;
    Ptrs ps = scan_ptrs(p);
    if constexpr (DK == DV && DK <= 128) {
        // few long chains: cut the sequences into G segments, get every segment's start state from a first pass
        // (k_scan_state, k_seg_combine), then run the scan below over the segments side by side
        const int G = segment_count(pb.N, pb.L, pb.H, DK, DV, DV / scan_vblock_cols((int)sizeof(T), DK, DV), pb.cu != nullptr);
        if (G > 1 && p.Sin) {
            sm.N = pb.N * G; sm.L = pb.L / G; sm.ncd = sm.L / C;
            DN_LAUNCH_SCAN(k_scan_state, DIR_BWD, 2, sm, pb.H, ps, half_);
            const CombineArgs ca{p.Mseg, p.Nseg, p.S0, p.Sin, p.ST, nullptr, nullptr, nullptr, nullptr, G, pb.H, 0};
            DN_LAUNCH_NT((k_seg_combine<DK, DV>), dim3(pb.N * pb.H, DV / kCombineCols, 1), kCombineThreads, (CombineSmem<DK, DV>::bytes), ca);
            ps.S0 = p.Sin; ps.ST = nullptr;
        }
    }
    if (pb.save) DN_LAUNCH_SCAN(k_scan_fwd_save, DIR_FWD, 1, sm, pb.H, ps);
    else DN_LAUNCH_SCAN(k_scan_fwd, DIR_FWD, 1, sm, pb.H, ps);
    return 0;
}

// the reverse scan of a backward pass, with the recompute scan in the same grid unless the forward pass left its tiles
template <typename T, int DK, int DV> int launch_bwd_scans(const Problem &pb, const SeqMap &sm, const Ptrs &p, const Ptrs &ps) {
    if (pb.save) DN_LAUNCH_SCAN(k_scan_bwd, DIR_BWD, 1, sm, pb.H, ps);
    else DN_LAUNCH_SCAN(k_scan_pair, DIR_BWD, 2, sm, pb.H, ps, half_);
    return 0;
}

template <typename T, int DK, int DV> int run_bwd(const Problem &pb, const Ptrs &p) {
    if (pb.N == 0) return 0;
    const SeqMap sm0 = make_map(pb);
    if (int e = launch_offsets(pb)) return e;
    Ptrs ps = scan_ptrs(p);
    // few long chains: the scans run over G segments of the sequences side by side (see k_scan_state)
    int G = 1;
    if constexpr (DK == DV && DK <= 128) G = segment_count_bwd(pb.N, pb.L, pb.H, DK, DV, DV / scan_vblock_cols((int)sizeof(T), DK, DV), pb.cu != nullptr);
    if (G > 1 && p.Sin && pb.chunks_ub) {
        if constexpr (DK == DV && DK <= 128) {
            SeqMap sm = sm0;
            sm.N = pb.N * G; sm.L = pb.L / G; sm.ncd = sm.L / C;
            if (pb.save) { // the forward pass left its tiles and the segments' transition matrices
                DN_LAUNCH_SCAN(k_scan_bwd_state, DIR_BWD, 1, sm, pb.H, ps);
                const CombineArgs ca{p.Mseg, nullptr, nullptr, nullptr, nullptr, p.Rseg, p.dST, p.dSout, p.dS0, G, pb.H, 1};
                DN_LAUNCH_NT((k_seg_combine<DK, DV>), dim3(pb.N * pb.H, DV / kCombineCols, 1), kCombineThreads, (CombineSmem<DK, DV>::bytes), ca);
            } else {
                if (int e = launch_prep<T, DK, DV>(pb, sm0, p)) return e;
                DN_LAUNCH_SCAN(k_scan_state, DIR_BWD, 3, sm, pb.H, ps, half_);
                const CombineArgs ca{p.Mseg, p.Nseg, p.S0, p.Sin, nullptr, p.Rseg, p.dST, p.dSout, p.dS0, G, pb.H, 0};
                DN_LAUNCH_NT((k_seg_combine<DK, DV>), dim3(pb.N * pb.H, DV / kCombineCols, 2), kCombineThreads, (CombineSmem<DK, DV>::bytes), ca);
                ps.S0 = p.Sin;
            }
            ps.dST = p.dSout; ps.dS0 = nullptr;
            if (int e = launch_bwd_scans<T, DK, DV>(pb, sm, p, ps)) return e;
        }
    } else {
        // kept tiles: T, Ut and the chunk-initial states are the forward pass's, only the reverse scan is left; otherwise both
        // scans of the backward pass as one grid: reverse scan first, recompute scan behind it
        if (!pb.save && pb.chunks_ub) if (int e = launch_prep<T, DK, DV>(pb, sm0, p)) return e;
        if (int e = launch_bwd_scans<T, DK, DV>(pb, sm0, p, ps)) return e;
    }
    const SeqMap &sm = sm0;
    if (pb.chunks_ub) {
        const long tiles = (long)pb.chunks_ub * pb.H, slots = (long)pb.num_cus * local_wpc<T, DK, DV>();
        const dim3 gpers((unsigned)(tiles < slots ? tiles : slots)); // persistent: as many workgroups as the chip holds
        constexpr size_t lds = LocalLds<T, DK, DV>;
        if (p.g) DN_LAUNCH_NT((k_bwd_local<T, DK, DV, VAR_GATED>), gpers, NTC, lds, sm, pb.H, p, pb.chunks_ub);
        else if (p.pro) DN_LAUNCH_NT((k_bwd_local<T, DK, DV, VAR_PROLOGUE>), gpers, NTC, lds, sm, pb.H, p, pb.chunks_ub);
        else DN_LAUNCH_NT((k_bwd_local<T, DK, DV, VAR_PLAIN>), gpers, NTC, lds, sm, pb.H, p, pb.chunks_ub);
        if (p.dv_out) { // the inputs have been read
            const long words = (long)(pb.cu ? 1 : pb.N) * pb.L * pb.H * DV * (long)sizeof(T) / 4; // (rows are at least 64 bytes)
            DN_LAUNCH(k_state_copy, dim3((unsigned)((words + 4 * NTHR - 1) / (4 * NTHR))), 0, static_cast<float *>(p.dv_out), static_cast<const float *>(p.dv), words);
        }
    }
    return 0;
}

#define DN_INSTANTIATE(T, DK, DV)                                        \
    template int run_fwd<T, DK, DV>(const Problem &, const Ptrs &);      \
    template int run_bwd<T, DK, DV>(const Problem &, const Ptrs &);      \
    template size_t max_lds_bytes<T, DK, DV>();

} // namespace dn
