// The kernels of the chunkwise DeltaNet forward/backward (gfx950), templated on the element
// type T (float: fp32 MFMA; bf16: bf16 MFMA with fp32 accumulation) and the head dims.
//
//   k_wy_prep    per chunk            A = tril(diag(beta) K K^T,-1); X = (I+A)^-1; T = X diag(beta)   (Eq. 10)
//   k_scan_fwd   per chain x v-block  serial over chunks: Ut = T (V - K S); P = tril(Q K^T); O = Q S + P Ut; S += K^T Ut  (Eq. 8-9, 11)
//   k_scan_pair  per chain x v-block  backward: the state-recompute scan (stores chunk-initial S and Ut) and the reverse
//                                     scan (dUt = P^T dO + K dS'; dV = T^T dUt; dS = dS' + Q^T dO - K^T dV) as one grid (dn_scan.hpp)
//   k_scan_fwd_save / k_scan_bwd      the forward scan that also stores what the recompute scan would, and the reverse
//                                     scan alone, for a backward pass that keeps the forward pass's tiles
//   k_bwd_local  per chunk            given S, dS', Ut, dV: the chunk-local rest of the adjoint, dQ, dK, dbeta (dn_chunk_bf16.hpp, dn_chunk_local.hpp)
//
// State S is [d_k][d_v] (orientation of the paper's pseudocode listing), fp32 in registers.
#pragma once
#include "dn_device.hpp"
#include "dn_host.hpp"

namespace dn {

constexpr int cmax(int a, int b) { return a > b ? a : b; }
// Kernel variants (a compile-time template argument, so that each carries only its own registers):
// the plain delta rule; the gated rule; the plain rule with the layer's prologue (q, k = SiLU(x) /
// ||SiLU(x)||_2 of section 3.3, beta = sigmoid(b) of section 2.2).  For the prologue k_wy_prep maps q
// and k once and leaves them in the workspace for the scans, which run the plain variant on them;
// k_bwd_local reads the mapped tiles too and sends the gradients back through the map on
// the way out, so dq, dk never reach HBM in the mapped coordinates.
enum { VAR_PLAIN = 0, VAR_GATED = 1, VAR_PROLOGUE = 2 };
// |beta| below this counts as a masked token in the backward pass: dbeta is not taken from a quotient by it (its square, and
// products of its size, stay far inside fp32 above it)
constexpr float kTinyBeta = 0x1p-40f;
constexpr size_t align16(size_t x) { return (x + 15) & ~size_t(15); }

} // namespace dn

#include "dn_scan.hpp"

namespace dn {

// ---------------------------------------------------------------------------------------------
// Packed layout, one workgroup.  The caller's offsets are first bounded: cus[n] = the running maximum of cu[0..n], held
// inside [0, L].  For a valid array (0 = cu[0] <= cu[1] <= ... <= cu[N] = L) that is the array itself; a malformed one that
// no host copy was there to reject becomes some non-decreasing sequence inside the tensors, so that every row index and
// every workspace tile the other kernels derive from it stays in bounds (the results are then meaningless).  Every other
// kernel reads cus, never cu.  Then the per-sequence chunk-count prefix coff[n] = sum_{m<n} ceil(len_m / C) and, behind
// it, order[i] = the i-th longest sequence (ties by index): the chain-serial kernels start the long chains first, so
// that the short ones fill the tail (up to kMaxOrdered sequences; more than that balance by themselves and keep their order).
// Workspace: coff [N + 1], order [N], cus [N + 1].
constexpr int kMaxOrdered = 512;
static __global__ void k_chunk_offsets(const int32_t *cu_in, int N, int L, int32_t *coff) {
    int32_t *order = coff + N + 1, *cu = order + N;
    __shared__ int part[NTHR];
    const int tid = threadIdx.x;
    {
        const int per1 = (N + 1 + NTHR - 1) / NTHR, lo1 = tid * per1, hi1 = min(N + 1, lo1 + per1);
        int m = 0;
        for (int n = lo1; n < hi1; ++n) m = max(m, min(cu_in[n], L));
        part[tid] = m;
        __syncthreads();
        if (tid == 0) {
            int run = 0;
            for (int i = 0; i < NTHR; ++i) { const int t = part[i]; part[i] = run; run = max(run, t); }
        }
        __syncthreads();
        int run = part[tid];
        for (int n = lo1; n < hi1; ++n) { run = max(run, min(cu_in[n], L)); cu[n] = run; }
        __syncthreads();
    }
    if (N <= kMaxOrdered) {
        for (int n = threadIdx.x; n < N; n += NTHR) {
            const int len = cu[n + 1] - cu[n];
            int rank = 0;
            for (int m = 0; m < N; ++m) {
                const int lm = cu[m + 1] - cu[m];
                rank += (lm > len) || (lm == len && m < n);
            }
            order[rank] = n;
        }
    } else {
        for (int n = threadIdx.x; n < N; n += NTHR) order[n] = n;
    }
    const int per = (N + NTHR - 1) / NTHR;
    const int lo = tid * per, hi = min(N, lo + per);
    int s = 0;
    for (int n = lo; n < hi; ++n) s += (cu[n + 1] - cu[n] + C - 1) / C;
    part[tid] = s;
    __syncthreads();
    if (tid == 0) {
        int run = 0;
        for (int i = 0; i < NTHR; ++i) { int t = part[i]; part[i] = run; run += t; }
        coff[N] = run;
    }
    __syncthreads();
    int run = part[tid];
    for (int n = lo; n < hi; ++n) { coff[n] = run; run += (cu[n + 1] - cu[n] + C - 1) / C; }
}

// plain copy of 32-bit words (src null: zeros): final_state of a pass over no tokens at all, which is the initial state or zero;
// dv from the workspace to a buffer that was also an input
static __global__ void k_state_copy(float *dst, const float *src, long count) {
    for (long i = (long)blockIdx.x * blockDim.x + threadIdx.x; i < count; i += (long)gridDim.x * blockDim.x) dst[i] = src ? src[i] : 0.f;
}

// =============================================================================================
// k_wy_prep: per chunk, T = (I + tril(diag(beta) K K^T, -1))^-1 diag(beta) (Eq. 10).
// W = T K and U = T V (Eq. 11) are never formed, the scans multiply V - K S by T: 8 KB per chunk
// where W and U are 32 KB.
// A chain of short serial stages per workgroup: what counts is how many are resident (eight per CU; K unpadded beyond 16 bytes a
// row, the inverse in K's bytes and without scratch) and the LDS instructions of the inverse.  Against the form with the merges
// on the vector ALU (six per CU, chunks fastest): 16 384 tokens of width 2048, d = 128 34 -> 25 us (100 MB, 4 TB/s), d = 64
// 59 -> 43 us, d = 256 30 -> 24 us.  (The Gram product is formed transposed, so that a lane's four elements of A are neighbours and have one beta: with a
// read of beta and a store for each of the 16 the kernel took 27.7 us for 26.6, at d = 64 39.1 for 37.0, on 1 x 1000 tokens 8.1 for 7.4.)  The prologue variant (two tiles mapped on the way, four per CU) takes 64 us for 300 MB.
template <typename T, int DK, int DV> struct PrepSmem {
    static constexpr int LD = ldc<T>(DK), LF = C + 4;
    // K while the Gram product runs, then the fp32 matrix that is inverted in place
    static constexpr size_t oK = 0, oX = 0;
    static constexpr size_t oBeta = align16(cmax(sizeof(T) * C * LD, sizeof(float) * C * LF));
    static constexpr size_t bytes = oBeta + sizeof(float) * C;
};

// (bf16 up to d_k = 128: held to the registers of eight workgroups per CU, which is what its LDS allows, with the prologue's registers
// four, at d_k = 64 five: with four the forward pass took 144.6 us for 141 there, 8 x 2048 tokens of 32 heads; the other instantiations would spill under such a cap)
template <typename T, int DK, bool PRO> struct PrepWaves { static constexpr int lo = (sizeof(T) == 2 && DK <= 128) ? (PRO ? (DK > 64 ? 4 : 5) : 8) : 1, hi = lo > 1 ? lo : 8; };
template <typename T, int DK, int DV, bool PRO>
__global__ __launch_bounds__(NTHR) __attribute__((amdgpu_waves_per_eu(PrepWaves<T, DK, PRO>::lo, PrepWaves<T, DK, PRO>::hi))) void k_wy_prep(SeqMap sm, int H, Ptrs p) {
    using SM = PrepSmem<T, DK, DV>;
    extern __shared__ __align__(16) unsigned char smem[];
    T *sK = reinterpret_cast<T *>(smem + SM::oK);
    float *sX = reinterpret_cast<float *>(smem + SM::oX);
    float *sBeta = reinterpret_cast<float *>(smem + SM::oBeta);

    // heads run fastest: the workgroups in flight then read whole rows of k between them (a head's part of a row is 128 to 512
    // bytes; many of those at a stride of a row is a pattern that HBM serves at about half its rate)
    int n, ic;
    const int h = (int)(blockIdx.x % (unsigned)H);
    if (!sm.chunk((int)(blockIdx.x / (unsigned)H), n, ic)) return;
    int t0, len, cb;
    sm.seq(n, t0, len, cb);
    const int tid = threadIdx.x, wave = tid >> 6;
    const int nvalid = min(C, len - ic * C);
    const long row0 = (long)t0 + (long)ic * C;
    const long tile = ((long)(cb + ic) * H + h);
    const int mi = wave >> 1, ni = wave & 1; // this wave's 32 x 32 tile of the C x C matrices
    const bool upper = mi == 0 && ni == 1;

    {
        TileRegs<T, C, DK> kr;
        // (prologue variant: the raw tiles are not needed again before the chunk kernel; not kept in the caches, they leave those to the mapped ones,
        // which the scan reads next: forward scan that keeps its tiles 95.8 -> 92.4 us, 8 x 2048 tokens of 16 heads of 128.  At d_k = 64 a batch
        // whose inputs fit the caches loses more by it: forward pass on 5 x 1500 tokens of 32 heads, run repeatedly, 73.3 us with the raw tiles
        // kept, 79.2 without, on new inputs 77.2 either way)
        constexpr int kAuxRaw = PRO && DK > 64 ? kAuxOnce : kAuxKeep;
        kr.template load_aux<kAuxRaw>((const T *)p.k + (row0 * H + h) * DK, (long)H * DK, nvalid, threadIdx.x);
        if constexpr (PRO) { // prologue variant: q and k arrive before the feature map of section 3.3
            TileRegs<T, C, DK> qr;
            qr.template load_aux<kAuxRaw>((const T *)p.q + (row0 * H + h) * DK, (long)H * DK, nvalid, threadIdx.x);
            float inv[TileRegs<T, C, DK>::NIT];
            kr.feature_map(inv);
            kr.store_global((T *)p.Km + (row0 * H + h) * DK, (long)H * DK, nvalid);
            qr.feature_map(inv);
            qr.store_global((T *)p.Qm + (row0 * H + h) * DK, (long)H * DK, nvalid);
        }
        kr.store(sK, SM::LD);
    }
    if (tid < C) {
        float b = tid < nvalid ? to_f32(((const T *)p.beta)[(row0 + tid) * H + h]) : 0.f;
        if (PRO) b = tid < nvalid ? sigmoid_f32(b) : 0.f; // ... and beta before the sigmoid
        sBeta[tid] = b;
    }
    if (p.g && tid < C) {
        // Gated variant: with the running decay exp(g_1 + ... + g_i) within the chunk (rows past the end keep the last
        // value), the state divided by it follows the plain delta rule on equally divided values, so the other kernels
        // only rescale rows with gamma_i and 1 / gamma_i; T does not depend on the gate.  The table holds the decay
        // relative to the chunk's geometric middle, gamma_i = exp(g_1 + ... + g_i - (g_1 + ... + g_C) / 2): both
        // gamma_i and 1 / gamma_i then stay within exp(+-sum|g| / 2), which doubles the decay per chunk that fp32 holds.
        // The chain scans move the state into these coordinates when a chunk begins (factor gamma_C, which in them is
        // also the decay from the chunk's start to its middle) and out of them when it ends (gamma_C again).
        float cs = tid < nvalid ? p.g[(row0 + tid) * H + h] : 0.f;
#pragma unroll
        for (int d = 1; d < 64; d <<= 1) {
            const float up = __shfl_up(cs, d);
            if (tid >= d) cs += up;
        }
        const float half = 0.5f * __shfl(cs, C - 1);
        p.gam[tile * 2 * C + tid] = __expf(cs - half);
        p.gam[tile * 2 * C + C + tid] = __expf(half - cs);
    }
    lds_barrier();
    f32x16 g = zero16();
    if (!upper) mma<DK, false, false, T, true, sizeof(T) == 2 ? 2 : 0>(g, sK + 32 * ni * SM::LD, SM::LD, sK + 32 * mi * SM::LD, SM::LD); // (K K^T)^T
    lds_barrier(); // K is dead from here on; its bytes take the fp32 matrix
    if (!upper) { // A = tril(diag(beta) K K^T, -1): a lane has 16 columns j of its row i, four at a time next to each other
        const int lane = tid & 63, i = 32 * mi + (lane & 31), below = i - 32 * ni - 4 * (lane >> 5); // i - j of element 0
        const float b = sBeta[i];
        float *row = sX + i * SM::LF + 32 * ni + 4 * (lane >> 5);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            f32x4 a;
#pragma unroll
            for (int u = 0; u < 4; ++u) a[u] = below > 8 * e + u ? b * g[4 * e + u] : 0.f;
            *reinterpret_cast<f32x4 *>(row + 8 * e) = a;
        }
    }
    lds_barrier();
    tri_inverse_64(sX, SM::LF);
    // T = X diag(beta), converted and written 16 bytes at a time (X21 stands in the upper right block).  The diagonal, which is beta,
    // is left out: the scans put that term in from numbers that have not been rounded.  Every wave clears it in the 16 rows that it
    // then reads, and the zero block is selected by piece: comparisons and selections per element, in all 32 wavefronts of a CU, took 29.6 us
    // for 26.6, at d = 64 41.2 for 37.3 (8 x 2048 tokens of width 2048).
    constexpr int VEC = El<T>::VEC, SEGS = C / VEC, RPW = 64 / SEGS; // rows per wave and round of the loop below
    if ((tid & 63) < 16) {
        const int r = RPW * (wave + NTHR / 64 * ((tid & 63) / RPW)) + (tid & 63) % RPW;
        sX[r * SM::LF + r] = 0.f;
    }
    wave_exchange();
    for (int e = tid; e < C * SEGS; e += NTHR) {
        const int i = e / SEGS, j0 = (e % SEGS) * VEC;
        const float *x = sX + (i >= 32 && j0 < 32 ? (i - 32) * SM::LF + 32 + j0 : i * SM::LF + j0);
        const bool zero = i < 32 && j0 >= 32;
        alignas(16) T tv[VEC];
#pragma unroll
        for (int u = 0; u < VEC; ++u) tv[u] = from_f32<T>(x[u] * sBeta[j0 + u]);
        const u32x4 piece = zero ? u32x4{0, 0, 0, 0} : *reinterpret_cast<const u32x4 *>(tv);
        __builtin_nontemporal_store(piece, reinterpret_cast<u32x4 *>((T *)p.Tm + tile * C * C + i * C + j0));
    }
}

// =============================================================================================
// The chain-serial kernels (dn_scan.hpp): NCW chain waves of 16 state columns each and four or eight helper waves per workgroup
template <typename T, int DK, int DV, bool GATED, int NCW>
__global__ __launch_bounds__((kScanThreads<T, DK, DIR_FWD, NCW>)) void k_scan_fwd(SeqMap sm, int H, Ptrs p) {
    scan_fwd_body<T, DK, DV, SCAN_OUT, GATED, NCW>(sm, H, p, blockIdx.x);
}
template <typename T, int DK, int DV, bool GATED, int NCW>
__global__ __launch_bounds__((kScanThreads<T, DK, DIR_FWD, NCW>)) void k_scan_fwd_save(SeqMap sm, int H, Ptrs p) {
    scan_fwd_body<T, DK, DV, SCAN_BOTH, GATED, NCW>(sm, H, p, blockIdx.x);
}

// A forward pass over few, long chains leaves most CUs idle.  Every stretch of a chain acts on the state as an
// affine map S_out = M S_in + N (M = the product of the chunks' (I - K^T T K), d_k x d_k; N = what the stretch writes
// starting from zero; Eq. 8), so the sequence is cut into G segments that are scanned side by side:
//   k_scan_state   per segment, both in one grid: N (the scan from a zero state) and M (the same scan on v = 0
//                  starting from the identity; needs d_v = d_k), final states only
//   k_seg_combine  per chain: S_in of every segment by S <- M_g S + N_g, in fp32 on the matrix cores
//   k_scan_fwd     per segment, from its S_in: the outputs
// `sm` describes the segments as sequences (dense layout: [B, L] viewed as [B G, L / G]); `half` = workgroups per pass.
// The backward pass is cut the same way: the gradient with respect to a segment's start state is
// M^T (gradient with respect to its end state) + R, R = the reverse scan of the segment from a zero gradient; a grid of
// three parts adds that pass (k_scan_state), a grid of one part runs it alone (k_scan_bwd_state).
template <typename T, int DK, int DV, bool GATED, int NCW>
__global__ __launch_bounds__((kScanThreads<T, DK, DIR_BWD, NCW>)) void k_scan_state(SeqMap sm, int H, Ptrs p, int half) {
    Ptrs ps = p;
    ps.S0 = nullptr;
    const int part = (int)blockIdx.x / half, bid = (int)blockIdx.x - part * half;
    if (part == 2) {
        ps.dST = nullptr; ps.dS0 = p.Rseg;
        scan_bwd_body<T, DK, DV, GATED, true, NCW>(sm, H, ps, bid);
        return;
    }
    if (part == 0) { ps.unit_state = 0; ps.ST = p.Nseg; }
    else { ps.unit_state = 1; ps.ST = p.Mseg; }
    scan_fwd_body<T, DK, DV, SCAN_STATE, GATED, NCW>(sm, H, ps, bid);
}
template <typename T, int DK, int DV, bool GATED, int NCW>
__global__ __launch_bounds__((kScanThreads<T, DK, DIR_BWD, NCW>)) void k_scan_bwd_state(SeqMap sm, int H, Ptrs p) {
    Ptrs ps = p;
    ps.dST = nullptr; ps.dS0 = p.Rseg;
    scan_bwd_body<T, DK, DV, GATED, true, NCW>(sm, H, ps, blockIdx.x);
}

// S_in(0) = the caller's initial state (or zero); S_in(g + 1) = M_g S_in(g) + N_g; the state after the last segment is
// the final state.  Backward (blockIdx.z = 1): D(G) = the caller's gradient with respect to the final state (or zero);
// every segment's end gradient dSout(g) = D(g + 1), D(g) = M_g^T D(g + 1) + R_g; D(0) is the gradient with respect to the
// initial state.  One workgroup per (chain, block of 16 state columns, direction): the columns evolve independently.
// fp32 on the matrix cores; the next segment's M and N (R) tile travel from global memory while the current product runs.
// A wave owns 16 rows of the product, in 16 x 16 x 4 matrix instructions: DK / 4 dependent ones a segment (1 K cycles at d = 128).
constexpr int kCombineCols = 16, kCombineThreads = 512;
template <int DK, int DV> struct CombineSmem {
    static constexpr int LM = DK + 4, LSB = 16 + 4;
    static constexpr size_t oM = 0, oS = sizeof(float) * DK * LM, bytes = oS + sizeof(float) * DK * LSB;
};
struct CombineArgs {
    const float *Mseg, *Nseg, *S0; // forward: per-segment N, the caller's initial state (may be null)
    float *Sin, *ST;               // forward outputs: start state per segment, final state (may be null)
    const float *Rseg, *dST;       // backward: per-segment R, the caller's final-state gradient (may be null)
    float *dSout, *dS0;            // backward outputs: end gradient per segment, initial-state gradient (may be null)
    int G, H, first_dir;           // grid.z directions run from first_dir: 0 = forward, 1 = backward
};
template <int DK, int DV>
__global__ __launch_bounds__(kCombineThreads) void k_seg_combine(CombineArgs a) {
    using SM = CombineSmem<DK, DV>;
    constexpr int NT = kCombineThreads, NB = kCombineCols;
    static_assert(DK % 16 == 0 && DK / 16 <= NT / 64, "one tile of 16 rows per wave");
    extern __shared__ __align__(16) unsigned char smem[];
    float *sM = reinterpret_cast<float *>(smem + SM::oM), *sS = reinterpret_cast<float *>(smem + SM::oS);
    const int chain = blockIdx.x, b = chain / a.H, h = chain - b * a.H, c0 = NB * blockIdx.y;
    const bool bwd = (int)blockIdx.z + a.first_dir == 1;
    const int tid = threadIdx.x, wave = tid >> 6, j = tid & 15, g4 = 4 * ((tid & 63) >> 4);
    const bool act = wave < DK / 16;
    const int row0 = 16 * wave + g4; // the first of this lane's four rows, column j
    const float *init = bwd ? a.dST : a.S0, *add = bwd ? a.Rseg : a.Nseg;
    float *start = bwd ? a.dSout : a.Sin, *last = bwd ? a.dS0 : a.ST;
    auto seg_of = [&](int i) __attribute__((always_inline)) { return ((long)(b * a.G + (bwd ? a.G - 1 - i : i)) * a.H + h); };
    TileRegs<float, DK, DK, NT> mreg;
    f32x4 nreg = {0.f, 0.f, 0.f, 0.f}, cur = nreg; // cur: the current value of this lane's rows
    auto request = [&](int i) __attribute__((always_inline)) { // M and the additive tile of step i, into registers
        const long seg = seg_of(i);
        mreg.load(a.Mseg + seg * DK * DK, DK, DK);
        if (act)
#pragma unroll
            for (int e = 0; e < 4; ++e) nreg[e] = add[(seg * DK + row0 + e) * DV + c0 + j];
    };
    request(0);
    if (act && init)
#pragma unroll
        for (int e = 0; e < 4; ++e) cur[e] = init[((long)chain * DK + row0 + e) * DV + c0 + j];
    for (int i = 0; i < a.G; ++i) {
        const long seg = seg_of(i);
        if (act) // this segment starts from (backward: ends with) the current value
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                start[(seg * DK + row0 + e) * DV + c0 + j] = cur[e];
                sS[(row0 + e) * SM::LSB + j] = cur[e];
            }
        mreg.store(sM, SM::LM);
        f32x4 acc[2] = {nreg, {0.f, 0.f, 0.f, 0.f}};
        lds_barrier(); // (LDS only: the requests and stores in flight are not waited for)
        if (i + 1 < a.G) request(i + 1);
        if (act) {
#pragma unroll
            for (int k = 0; k < DK; k += 16) { // lane group g feeds the contraction indices k + 4 g + e in step e
                f32x4 m;
                if (bwd)
#pragma unroll
                    for (int e = 0; e < 4; ++e) m[e] = sM[(k + g4 + e) * SM::LM + 16 * wave + j]; // M^T D: down the rows of M
                else m = *reinterpret_cast<const f32x4 *>(sM + (16 * wave + j) * SM::LM + k + g4);
#pragma unroll
                for (int e = 0; e < 4; ++e) acc[e & 1] = mfma16(acc[e & 1], m[e], sS[(k + g4 + e) * SM::LSB + j]);
            }
            cur = acc[0] + acc[1];
        }
        lds_barrier(); // every wave has read the old value
    }
    if (last && act)
#pragma unroll
        for (int e = 0; e < 4; ++e) last[((long)chain * DK + row0 + e) * DV + c0 + j] = cur[e];
}

// The backward pass's two scans in one launch.  They do not depend on each other (the recompute
// scan needs T; the reverse scan needs T and P^T), so the first half of the grid runs the reverse
// scan and the second half the recompute scan: a CU picks up one of each with no kernel boundary
// in between.  `half` = workgroups per scan.
template <typename T, int DK, int DV, bool GATED, int NCW>
__global__ __launch_bounds__((kScanThreads<T, DK, DIR_BWD, NCW>)) void k_scan_pair(SeqMap sm, int H, Ptrs p, int half) {
    if ((int)blockIdx.x < half) scan_bwd_body<T, DK, DV, GATED, false, NCW>(sm, H, p, blockIdx.x);
    else scan_fwd_body<T, DK, DV, SCAN_STORE, GATED, NCW>(sm, H, p, blockIdx.x - half);
}
// the reverse scan alone, for a backward pass that finds the forward scan's tiles already in the workspace
template <typename T, int DK, int DV, bool GATED, int NCW>
__global__ __launch_bounds__((kScanThreads<T, DK, DIR_BWD, NCW>)) void k_scan_bwd(SeqMap sm, int H, Ptrs p) {
    scan_bwd_body<T, DK, DV, GATED, false, NCW>(sm, H, p, blockIdx.x);
}

// =============================================================================================
// The chunk-parallel backward kernel (dn_chunk_bf16.hpp, dn_chunk_local.hpp).  Workgroups are persistent: each walks over
// (chunk, head) tiles with a grid stride.
constexpr int NTC = 512, NWC = 8;

struct TileIter { // grid-stride walk over (global chunk id, head) tiles
    int id, total, H;
    __device__ TileIter(int chunks_total, int H_) : id(blockIdx.x), total(chunks_total * H_), H(H_) {}
    __device__ bool valid() const { return id < total; }
    __device__ void next() { id += gridDim.x; }
    __device__ int gid() const { return id / H; }
    __device__ int head() const { return id % H; }
};
struct TilePos { int nvalid, h; long row0, tile; bool ok; };
__device__ inline TilePos tile_pos(const SeqMap &sm, int H, int gid, int h) {
    TilePos tp;
    int n, ic, t0, len, cb;
    tp.ok = sm.chunk(gid, n, ic);
    tp.h = h; tp.nvalid = 0; tp.row0 = 0; tp.tile = 0;
    if (tp.ok) {
        sm.seq(n, t0, len, cb);
        tp.nvalid = min(C, len - ic * C);
        tp.row0 = (long)t0 + (long)ic * C;
        tp.tile = (long)(cb + ic) * H + h;
    }
    return tp;
}

} // namespace dn
