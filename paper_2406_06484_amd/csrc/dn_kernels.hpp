// The kernels of the chunkwise DeltaNet forward/backward (gfx950), templated on the element
// type T (float: fp32 MFMA; bf16: bf16 MFMA with fp32 accumulation) and the head dims.
//
//   k_wy_prep    per chunk            A = tril(diag(beta) K K^T,-1); X = (I+A)^-1; T = X diag(beta)   (Eq. 10)
//   k_scan_fwd   per chain x v-block  serial over chunks: W = T K, U = T V (Eq. 11); Ut = U - W S; P = tril(Q K^T); O = Q S + P Ut; S += K^T Ut  (Eq. 8-9)
//   k_scan_pair  per chain x v-block  backward: the state-recompute scan (stores chunk-initial S and Ut) and the reverse
//                                     scan (dUt = P^T dO + K dS'; dV = T^T dUt; dS = dS' + Q^T dO - W^T dUt) as one grid
//   k_scan_fwd_save / k_scan_bwd      the forward scan that also stores what the recompute scan would, and the reverse
//                                     scan alone, for a backward pass that keeps the forward pass's tiles
//   k_bwd_local  per chunk            given S, dS', Ut, dV: the chunk-local rest of the adjoint, dQ, dK, dbeta (dn_chunk_local.hpp)
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
// and k once and leaves them in the workspace for the scans, which run the plain variant on them (the reverse scan
// that stores dV has one of its own, see scan_bwd_body);
// k_bwd_local reads the mapped tiles too and sends the gradients back through the map on
// the way out, so dq, dk never reach HBM in the mapped coordinates.
enum { VAR_PLAIN = 0, VAR_GATED = 1, VAR_PROLOGUE = 2 };
// |beta| below this counts as a masked token in the backward pass: dbeta is not taken from a quotient by it (its square, and
// products of its size, stay far inside fp32 above it)
constexpr float kTinyBeta = 0x1p-40f;
constexpr size_t align16(size_t x) { return (x + 15) & ~size_t(15); }

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
// W = T K and U = T V (Eq. 11) are rebuilt from T inside the scan kernels: T is 8 KB per chunk
// where W and U are 32 KB.
// A chain of short serial stages per workgroup: what counts is how many are resident (eight per CU; K unpadded beyond 16 bytes a
// row, the inverse in K's bytes and without scratch) and the LDS instructions of the inverse.  Against the form with the merges
// on the vector ALU (six per CU, chunks fastest): 16 384 tokens of width 2048, d = 128 34 -> 25 us (100 MB, 4 TB/s), d = 64
// 59 -> 43 us, d = 256 30 -> 24 us.  The prologue variant (two tiles mapped on the way, five per CU) takes 67 us for 300 MB as before.
template <typename T, int DK, int DV> struct PrepSmem {
    static constexpr int LD = ldc<T>(DK), LF = C + 4;
    // K while the Gram product runs, then the fp32 matrix that is inverted in place
    static constexpr size_t oK = 0, oX = 0;
    static constexpr size_t oBeta = align16(cmax(sizeof(T) * C * LD, sizeof(float) * C * LF));
    static constexpr size_t bytes = oBeta + sizeof(float) * C;
};

// (bf16 up to d_k = 128: held to the registers of eight workgroups per CU, which is what its LDS allows, five with the
// prologue's registers; the other instantiations would spill under such a cap)
template <typename T, int DK, bool PRO> struct PrepWaves { static constexpr int lo = (sizeof(T) == 2 && DK <= 128) ? (PRO ? 5 : 8) : 1, hi = lo > 1 ? lo : 8; };
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
        kr.template load_aux<kAuxKeep>((const T *)p.k + (row0 * H + h) * DK, (long)H * DK, nvalid, threadIdx.x);
        if constexpr (PRO) { // prologue variant: q and k arrive before the feature map of section 3.3
            TileRegs<T, C, DK> qr;
            qr.load((const T *)p.q + (row0 * H + h) * DK, (long)H * DK, nvalid);
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
    if (!upper) mma<DK, false, false, T, true, sizeof(T) == 2 ? 2 : 0>(g, sK + 32 * mi * SM::LD, SM::LD, sK + 32 * ni * SM::LD, SM::LD); // K K^T
    lds_barrier(); // K is dead from here on; its bytes take the fp32 matrix
    if (!upper)
        acc_each(g, [&](int r, int c, float &val) { // A = tril(diag(beta) K K^T, -1)
            const int i = 32 * mi + r, j = 32 * ni + c;
            sX[i * SM::LF + j] = j < i ? sBeta[i] * val : 0.f;
        });
    lds_barrier();
    tri_inverse_64(sX, SM::LF);
    // T = X diag(beta), converted and written 16 bytes at a time (X21 stands in the upper right block)
    constexpr int VEC = El<T>::VEC, SEGS = C / VEC;
    for (int e = tid; e < C * SEGS; e += NTHR) {
        const int i = e / SEGS, j0 = (e % SEGS) * VEC;
        const float *x = sX + (i >= 32 && j0 < 32 ? (i - 32) * SM::LF + 32 + j0 : i * SM::LF + j0);
        const bool zero = i < 32 && j0 >= 32;
        alignas(16) T tv[VEC];
#pragma unroll
        for (int u = 0; u < VEC; ++u) tv[u] = from_f32<T>(zero ? 0.f : x[u] * sBeta[j0 + u]);
        __builtin_nontemporal_store(*reinterpret_cast<const u32x4 *>(tv), reinterpret_cast<u32x4 *>((T *)p.Tm + tile * C * C + i * C + j0));
    }
}

// =============================================================================================
// The two chain-serial kernels.  One workgroup of 8 wavefronts owns one chain and BV = 64 columns (32: see VBlock)
// of the state; the state lives in accumulator registers, one 32 x 32 tile per wave.
// Waves 0..3 own the Ut / dUt tiles of the dependent chain; waves 4..7 have the lighter work between
// barriers and double as loaders: they request the next chunk's tiles and send most of the results
// out of LDS, so that the chain waves do not queue behind the CU's 64 B/clk vector-memory path in the
// intervals whose length they set (the one exception: the kept Ut / dUt tile of the previous step
// leaves through the chain waves in the last interval, where the loader waves are the busier side).
// W = T K (Eq. 11) is rebuilt per chunk from the 64 x 64 T.
// Workgroup ids are laid out so that the v-blocks of one chain land on the same XCD (ids are dealt
// round-robin over the 8 XCDs) and share its L2 for the Q, K, T tiles they both read.
constexpr int NTS = 512, NWS = 8, NTL = 256; // threads / waves of a scan workgroup; loader threads
// bf16 workgroups own 64 state columns; fp32 ones, and bf16 ones with d_k = 256, own 32, so that the
// tiles (whose rows are d_k long) still fit the 160 KB of LDS
template <typename T, int DV, int DK> struct VBlock {
    static constexpr int WANT = (sizeof(T) == 2 && DK <= 128) ? DN_VBLOCK_COLS : 32;
    static constexpr int BV = DV < WANT ? DV : WANT;
    static constexpr int NV = DV / BV;
    // what the scans of few chains take instead (see narrow_blocks in dn_launch.hpp)
    static constexpr int NARROW = BV == 64 ? 32 : BV;
};

__device__ inline bool chain_of_block(int bid, int nchains, int nv, int &chain, int &vbi) {
    const int xcd = bid & 7, slot = bid >> 3;
    vbi = slot % nv;
    chain = (slot / nv) * 8 + xcd;
    return chain < nchains;
}
__host__ inline int chain_grid(int nchains, int nv) { return ((nchains + 7) / 8) * 8 * nv; }

// Which tiles a scan wave owns.  State tile (sa, sb): rows 32*sa of d_k, cols 32*sb of the v-block.
// W tile: d_k block wk, chunk-row block wi.  Waves < U_TILES own U / Ut tile (ua, ub); waves 4..
// own the tile of O (forward) of the same shape.
template <int DK, int BV> struct ScanMap {
    static constexpr int NVT = BV / 32, NKT = DK / 32, S_TILES = NKT * NVT, U_TILES = 2 * NVT, W_TILES = 2 * NKT;
    static_assert(S_TILES <= NWS && U_TILES <= 4, "state tiling");
    int sa, sb, ua, ub;
    bool has_s, does_u, does_o;
    __device__ ScanMap(int wave) {
        sa = wave / NVT; sb = wave % NVT; has_s = wave < S_TILES;
        const int u = wave & 3;
        ua = u / NVT; ub = u % NVT;
        does_u = wave < U_TILES; does_o = wave >= 4 && u < U_TILES;
    }
};

// scan_fwd_body: MODE = SCAN_OUT writes O and the final state; SCAN_STORE (the backward's recompute pass)
// writes every chunk-initial state and Ut to the workspace instead of O; SCAN_BOTH (a forward pass whose
// backward pass will not recompute) does both; SCAN_STATE writes only the final state (the first pass of a
// forward pass that is split over segments of the sequence, see k_scan_state).
enum { SCAN_OUT = 0, SCAN_STORE = 1, SCAN_BOTH = 2, SCAN_STATE = 3 };
template <typename T, int DK, int DV, int BV> struct ScanFwdSmem {
    static constexpr int LQ = ldc<T>(DK), LK = ldn<T>(DK), LV = ldn<T>(BV), LS = ldc<T>(DK), LT = ldc<T>(C);
    static constexpr size_t oQ = 0;
    static constexpr size_t oK = oQ + align16(sizeof(T) * C * LQ);
    static constexpr size_t oV = oK + align16(sizeof(T) * C * LK);
    static constexpr size_t oW = oV + align16(sizeof(T) * C * LV);
    static constexpr size_t oST = oW + align16(sizeof(T) * C * LQ);
    static constexpr size_t oUT = oST + align16(sizeof(T) * BV * LS);
    static constexpr size_t szUT = align16(sizeof(T) * BV * LT);     // two Ut^T buffers, alternating by chunk parity
    static constexpr size_t oT = oUT + 2 * szUT;
    static constexpr size_t oP = oT + align16(sizeof(T) * C * LT);
    static constexpr size_t oStage = oP + align16(sizeof(T) * C * LT); // per-wave output staging tiles
    static constexpr int NSTG = ScanMap<DK, BV>::U_TILES; // only the output waves stage tiles
    static constexpr size_t oGam = oStage + NSTG * sizeof(T) * Stage<T>::ELEMS; // gated: gamma_i, 1 / gamma_i of the chunk
    static constexpr size_t bytes1 = oGam + sizeof(float) * 2 * C;
    // Where a second K tile and a second gamma table fit, the tiles of the next chunk move to LDS in the interval that
    // updates the state (which still reads the current K), and a chunk step takes three barrier intervals instead of four.
    static constexpr size_t szK = align16(sizeof(T) * C * LK);
    static constexpr bool kMerge = bytes1 + szK + sizeof(float) * 2 * C <= 160 * 1024;
    static constexpr size_t oK2 = bytes1, oGam2 = oK2 + szK;
    static constexpr size_t bytes = kMerge ? oGam2 + sizeof(float) * 2 * C : bytes1;
};

template <typename T, int DK, int DV, int MODE, int VAR, int BV>
__device__ __forceinline__ void scan_fwd_body(const SeqMap &sm, int H, const Ptrs &p, int bid) {
    using SM = ScanFwdSmem<T, DK, DV, BV>;
    static_assert(VAR != VAR_PROLOGUE, "the scans read q and k already mapped");
    constexpr bool GATED = VAR == VAR_GATED;
    constexpr bool OUT = MODE == SCAN_OUT || MODE == SCAN_BOTH, SAVE = MODE == SCAN_STORE || MODE == SCAN_BOTH;
    constexpr int NV = DV / BV;
    using Map = ScanMap<DK, BV>;
    constexpr int NWT = (Map::W_TILES + 3) / 4; // W tiles per chain wave
    extern __shared__ __align__(16) unsigned char smem[];
    T *stg = reinterpret_cast<T *>(smem + SM::oStage) + ((threadIdx.x >> 6) % SM::NSTG) * Stage<T>::ELEMS;
    T *sQ = reinterpret_cast<T *>(smem + SM::oQ);
    constexpr bool MERGE = SM::kMerge;
    T *sK0 = reinterpret_cast<T *>(smem + SM::oK), *sK1 = MERGE ? reinterpret_cast<T *>(smem + SM::oK2) : sK0;
    T *sV = reinterpret_cast<T *>(smem + SM::oV);
    T *sW = reinterpret_cast<T *>(smem + SM::oW);
    T *sST = reinterpret_cast<T *>(smem + SM::oST);
    T *sUT0 = reinterpret_cast<T *>(smem + SM::oUT), *sUT1 = reinterpret_cast<T *>(smem + SM::oUT + SM::szUT);
    T *sT = reinterpret_cast<T *>(smem + SM::oT);
    T *sP = reinterpret_cast<T *>(smem + SM::oP);
    float *sGam0 = reinterpret_cast<float *>(smem + SM::oGam), *sGam1 = MERGE ? reinterpret_cast<float *>(smem + SM::oGam2) : sGam0;
    constexpr bool gated = GATED; // compile-time, so the plain kernels carry none of the gate's registers
    // the gated kernels, and those with d_k = 256, request operand fragments in smaller batches: they have no registers to spare
    constexpr int MB = (GATED || MODE == SCAN_BOTH) ? 2 : (sizeof(T) == 4 ? 2 : (DK > 128 ? 4 : 0)); // SCAN_BOTH: the loader waves hold more
    // a workgroup's rows of V and O are whole 128-byte lines: non-temporal; with narrower column blocks a line is shared with
    // the neighbouring workgroup of the chain and keeps the default policy
    constexpr bool kWholeLines = BV * sizeof(T) >= 128;

    int chain, vbi;
    if (!chain_of_block(bid, sm.N * H, NV, chain, vbi)) return;
    int n = chain / H;
    const int h = chain - n * H, vb = vbi * BV;
    if (sm.order) { n = sm.order[n]; chain = n * H + h; } // packed: longest sequences first
    const int wave = threadIdx.x >> 6;
    int t0, len, cb;
    sm.seq(n, t0, len, cb);
    const int nchunks = (len + C - 1) / C;
    const Map m(wave);
    const bool loader = wave >= 4, does_o = OUT && m.does_o;
    const int lt = threadIdx.x - NTL; // index among the loader threads
    // waves 0..3 build the tiles (pmi, pni) = (0,0), (1,0), (1,1), (0,1) of P; the last one is all zero
    const int pmi = (wave == 1) | (wave == 2), pni = wave >> 1;

    f32x16 S = zero16();
    if (m.has_s && p.S0) {
        const float *src = p.S0 + (long)chain * DK * DV + vb;
        acc_each(S, [&](int r, int c, float &val) { val = src[(long)(32 * m.sa + r) * DV + 32 * m.sb + c]; });
    }
    if (MODE == SCAN_STATE && p.unit_state && m.has_s) // start from the identity: the final state is then the segment's transition matrix
        acc_each(S, [&](int r, int c, float &val) { val = (32 * m.sa + r == vb + 32 * m.sb + c) ? 1.f : 0.f; });
    // settle these loads here: otherwise the compiler keeps "state registers may still be in flight"
    // alive around the loop and drains the memory counter (and with it the prefetch) in every step
    __builtin_amdgcn_s_waitcnt(0x0F70); // vmcnt(0)

    struct Regs {
        TileRegs<T, C, DK, NTL> q, k;
        TileRegs<T, C, BV, NTL> v;
        TileRegs<T, C, C, NTL> t;
        float vs[TileRegs<T, C, BV, NTL>::NIT], gm; // gated: 1 / gamma of this lane's V rows; one entry of the gamma table
    } r;
    auto fetch_a = [&](int ic) __attribute__((always_inline)) {
        const int nvalid = min(C, len - ic * C);
        const long row0 = (long)t0 + (long)ic * C;
        const long tile = ((long)(cb + ic) * H + h);
        r.k.template load_aux<kAuxKeep>((const T *)p.k + (row0 * H + h) * DK, (long)H * DK, nvalid, lt);
        // (the transition-matrix pass of k_scan_state runs on v = 0: no row is valid)
        r.v.template load_aux<kWholeLines ? kAuxOnce : kAuxKeep>((const T *)p.v + (row0 * H + h) * DV + vb, (long)H * DV, (MODE == SCAN_STATE && p.unit_state) ? 0 : nvalid, lt);
        r.t.template load_aux<kAuxKeep>((const T *)p.Tm + tile * C * C, C, C, lt);
        if (gated) {
            r.v.load_row_factors(r.vs, p.gam + tile * 2 * C + C, lt);
            if (lt < 2 * C) r.gm = p.gam[tile * 2 * C + lt];
        }
    };
    auto fetch_b = [&](int ic) __attribute__((always_inline)) {
        const int nvalid = min(C, len - ic * C);
        const long row0 = (long)t0 + (long)ic * C;
        if (OUT) r.q.template load_aux<kAuxKeep>((const T *)p.q + (row0 * H + h) * DK, (long)H * DK, nvalid, lt);
    };
    // Everything that touches global memory is issued by the loader waves in one burst right after
    // the first barrier of a step: the loads for the next chunk, then the stores of what the previous
    // step left in LDS (its Ut^T, or its staged output tile).  The compiler drains the memory counter
    // when the loaded registers are moved to LDS at the top of the next step; by then all of it is a
    // full step old.
    auto flush_ut = [&](int icp, int t) __attribute__((always_inline)) { // Ut^T of chunk icp, still in LDS; t = 0 .. NTL - 1
        const long tile = ((long)(cb + icp) * H + h);
        copy_out<T, BV, C, NTL, true>((T *)p.Ut + (tile * DV + vb) * C, (icp & 1) ? sUT1 : sUT0, SM::LT, t);
    };
    auto flush_out = [&](int icp) __attribute__((always_inline)) { // this wave's staged output tile of chunk icp
        if (m.does_o)
            stage_flush<T, kWholeLines>(stg, (T *)p.o + (((long)t0 + (long)icp * C) * H + h) * DV + vb, (long)H * DV, 32 * m.ua, 32 * m.ub,
                           min(C, len - icp * C));
    };
    auto stash = [&](int par) __attribute__((always_inline)) { // fetched tiles of a chunk of parity `par`: registers -> LDS
        if (OUT) r.q.store(sQ, SM::LQ, lt);
        r.k.store(par ? sK1 : sK0, SM::LK, lt);
        if (gated) { // the chunk runs the plain rule on v_i / gamma_i
            r.v.scale_rows(r.vs);
            if (lt < 2 * C) (par ? sGam1 : sGam0)[lt] = r.gm;
        }
        r.v.store(sV, SM::LV, lt);
        r.t.store(sT, SM::LT, lt);
    };
    if (loader && nchunks > 0) { fetch_a(0); fetch_b(0); stash(0); }
    // gated: gamma at the end of the chunk, which rescales the state when the chunk is done; every wave
    // requests the next chunk's value one step ahead
    float gC = 1.f, gCn = 1.f;
    if (gated && nchunks > 0) {
        gCn = p.gam[((long)cb * H + h) * 2 * C + C - 1];
        S *= gCn; // into the first chunk's coordinates
    }
    for (int ic = 0; ic < nchunks; ++ic) {
        const long tile = ((long)(cb + ic) * H + h);
        T *sUT = (ic & 1) ? sUT1 : sUT0;
        T *sK = (ic & 1) ? sK1 : sK0;
        float *sGam = (ic & 1) ? sGam1 : sGam0;
        gC = gCn; // out of this chunk's coordinates when it ends (gC), and into the next one's (gCn)
        if (gated) gCn = ic + 1 < nchunks ? p.gam[(tile + H) * 2 * C + C - 1] : 1.f;
        if (!MERGE || ic == 0) {
            if (m.has_s) acc_to_lds_t<T>(sST, SM::LS, 32 * m.sa, 32 * m.sb, S);
        }
        lds_barrier();
        if (loader && ic + 1 < nchunks) fetch_a(ic + 1);
        if (MODE == SCAN_BOTH && loader) {
            // the chunk-initial state, kept for the backward pass, leaves in this interval (transposed, as it sits in
            // LDS); the previous chunk's Ut^T follows in the third one: both in one interval make it the longest
            copy_out<T, BV, DK, NTL, true>((T *)p.Sc + (tile * DV + vb) * DK, sST, SM::LS, lt);
        }
        f32x16 acc = zero16();
        if (!loader) {
            // What does not depend on the state, while the loader waves are busy with global memory.
            // Straight-line on purpose (full contraction length even where T's zero block makes half
            // of it idle, a masked all-zero P tile on wave 3): independent products in one basic
            // block are what lets the scheduler overlap one product's LDS and MFMA latency with the next.
            // (with more than two W tiles per wave, d_k = 256, the tiles are finished one at a time instead:
            // there are not enough registers to keep them all in flight)
            constexpr bool SEQ = GATED || NWT > 2;
            f32x16 w[NWT];
#pragma unroll
            for (int i = 0; i < NWT; ++i) { // W = T K (Eq. 11) as W^T = K^T T^T
                const int t = wave + 4 * i, wk = t % Map::NKT, wi = t / Map::NKT;
                w[i] = zero16();
                if (Map::W_TILES % 4 == 0 || t < Map::W_TILES) {
                    mma<C, true, false, T, SEQ, MB>(w[i], sK + 32 * wk, SM::LK, sT + 32 * wi * SM::LT, SM::LT);
                    if (NWT > 2) acc_to_lds_t<T>(sW, SM::LQ, 32 * wk, 32 * wi, w[i]);
                }
            }
            if (m.does_u) mma<C, false, true, T, SEQ, MB>(acc, sT + 32 * m.ua * SM::LT, SM::LT, sV + 32 * m.ub, SM::LV); // U = T V
            f32x16 pa = zero16();
            if (OUT) // P = tril(Q K^T), the causal intra-chunk scores of Eq. 9, as the tile (pni, pmi) of P^T
                mma<DK, false, false, T, SEQ, MB>(pa, sK + 32 * pni * SM::LK, SM::LK, sQ + 32 * pmi * SM::LQ, SM::LQ);
            if (NWT <= 2) {
#pragma unroll
                for (int i = 0; i < NWT; ++i) {
                    const int t = wave + 4 * i, wk = t % Map::NKT, wi = t / Map::NKT;
                    if (Map::W_TILES % 4 == 0 || t < Map::W_TILES) acc_to_lds_t<T>(sW, SM::LQ, 32 * wk, 32 * wi, w[i]);
                }
            }
            if (OUT) {
                acc_each(pa, [&](int r, int c, float &val) { if (32 * pni + r > 32 * pmi + c) val = 0.f; });
                acc_to_lds_t<T>(sP, SM::LT, 32 * pni, 32 * pmi, pa);
            }
        } else if (does_o) {
            // Q S, the inter-chunk part of Eq. 9: it needs only the state, so the output waves form it here,
            // where they would otherwise wait for the chain waves' products
            mma<DK, false, false, T, true, MB>(acc, sQ + 32 * m.ua * SM::LQ, SM::LQ, sST + 32 * m.ub * SM::LS, SM::LS);
        }
        lds_barrier();
        if (loader) {
            if (ic + 1 < nchunks) fetch_b(ic + 1);
            // the chunk-initial state leaves transposed, as it sits in LDS
            if (MODE == SCAN_STORE) copy_out<T, BV, DK, NTL, true>((T *)p.Sc + (tile * DV + vb) * DK, sST, SM::LS, lt);
            if (OUT && ic > 0) flush_out(ic - 1);
        }
        if (m.does_u) { // Ut = U - W S (inner term of Eq. 8-9)
            f32x16 ws = zero16();
            mma<DK, false, false, T, true, MB>(ws, sW + 32 * m.ua * SM::LQ, SM::LQ, sST + 32 * m.ub * SM::LS, SM::LS);
            acc -= ws;
            acc_to_lds_t<T>(sUT, SM::LT, 32 * m.ua, 32 * m.ub, acc);
        }
        lds_barrier();
        // the previous chunk's Ut^T leaves here, sent by the chain waves, which have no output tile to form in this interval
        if (SAVE && !loader && ic > 0) flush_ut(ic - 1, (int)threadIdx.x);
        if (does_o) { // O = Q S + P Ut (Eq. 9); the tile waits in this wave's staging area until the next step
            if (m.ua == 0) mma<32, false, false, T, true, MB>(acc, sP, SM::LT, sUT + 32 * m.ub * SM::LT, SM::LT);
            else mma<C, false, false, T, true, MB>(acc, sP + 32 * SM::LT, SM::LT, sUT + 32 * m.ub * SM::LT, SM::LT);
            if (gated) acc_each(acc, [&](int rr, int, float &val) { val *= sGam[32 * m.ua + rr]; }); // o_i = gamma_i o~_i
            acc_to_lds<T>(stg, Stage<T>::LD, 0, 0, acc);
        }
        if (m.has_s) mma<C, true, false, T, true, MB>(S, sK + 32 * m.sa, SM::LK, sUT + 32 * m.sb * SM::LT, SM::LT); // S += K^T Ut (Eq. 8)
        if (gated) { // from this chunk's coordinates to the state itself, then to the next chunk's (one factor at a time: their product may leave the fp32 range)
            S *= gC;
            S *= gCn;
        }
        if (MERGE) {
            // nothing read in this interval is written here: the state's LDS copy serves only the first two intervals of a
            // step, Q, V, T only the first, and the next K and gamma table go to the buffers of the other parity
            if (m.has_s && ic + 1 < nchunks) acc_to_lds_t<T>(sST, SM::LS, 32 * m.sa, 32 * m.sb, S);
        } else {
            lds_barrier();
        }
        // The next chunk's tiles move to LDS here, in the iteration that requested them: the wait the
        // compiler puts in front counts the stores issued after the loads and lets those stay in flight.
        if (loader && ic + 1 < nchunks) stash((ic + 1) & 1);
    }
    if (loader && nchunks > 0) {
        if (SAVE) flush_ut(nchunks - 1, lt);
        if (OUT) flush_out(nchunks - 1);
    }
    if ((OUT || MODE == SCAN_STATE) && p.ST && m.has_s) {
        float *dst = p.ST + (long)chain * DK * DV + vb;
        acc_each(S, [&](int r, int c, float &val) { dst[(long)(32 * m.sa + r) * DV + 32 * m.sb + c] = val; });
    }
}
template <typename T, int DK, int DV, int VAR, int BV>
__global__ __launch_bounds__(NTS) void k_scan_fwd(SeqMap sm, int H, Ptrs p) {
    scan_fwd_body<T, DK, DV, SCAN_OUT, VAR, BV>(sm, H, p, blockIdx.x);
}
template <typename T, int DK, int DV, int VAR, int BV>
__global__ __launch_bounds__(NTS) void k_scan_fwd_save(SeqMap sm, int H, Ptrs p) {
    scan_fwd_body<T, DK, DV, SCAN_BOTH, VAR, BV>(sm, H, p, blockIdx.x);
}

template <typename T, int DK, int DV, int VAR, bool STATE, int BV>
__device__ __forceinline__ void scan_bwd_body(const SeqMap &sm, int H, const Ptrs &p, int bid);

// A forward pass over few, long chains leaves most CUs idle.  Every stretch of a chain acts on the state as an
// affine map S_out = M S_in + N (M = the product of the chunks' (I - K^T W), d_k x d_k; N = what the stretch writes
// starting from zero; Eq. 8), so the sequence is cut into G segments that are scanned side by side:
//   k_scan_state   per segment, both in one grid: N (the scan from a zero state) and M (the same scan on v = 0
//                  starting from the identity; needs d_v = d_k), final states only
//   k_seg_combine  per chain: S_in of every segment by S <- M_g S + N_g, in fp32 on the matrix cores
//   k_scan_fwd     per segment, from its S_in: the outputs
// `sm` describes the segments as sequences (dense layout: [B, L] viewed as [B G, L / G]); `half` = workgroups per pass.
// The backward pass is cut the same way: the gradient with respect to a segment's start state is
// M^T (gradient with respect to its end state) + R, R = the reverse scan of the segment from a zero gradient; a grid of
// three parts adds that pass (k_scan_state), a grid of one part runs it alone (k_scan_bwd_state).
template <typename T, int DK, int DV, int VAR>
__global__ __launch_bounds__(NTS) void k_scan_state(SeqMap sm, int H, Ptrs p, int half) {
    Ptrs ps = p;
    ps.S0 = nullptr;
    const int part = (int)blockIdx.x / half, bid = (int)blockIdx.x - part * half;
    if (part == 2) {
        ps.dST = nullptr; ps.dS0 = p.Rseg;
        scan_bwd_body<T, DK, DV, VAR, true, VBlock<T, DV, DK>::BV>(sm, H, ps, bid);
        return;
    }
    if (part == 0) { ps.unit_state = 0; ps.ST = p.Nseg; }
    else { ps.unit_state = 1; ps.ST = p.Mseg; }
    scan_fwd_body<T, DK, DV, SCAN_STATE, VAR, VBlock<T, DV, DK>::BV>(sm, H, ps, bid);
}
template <typename T, int DK, int DV, int VAR>
__global__ __launch_bounds__(NTS) void k_scan_bwd_state(SeqMap sm, int H, Ptrs p) {
    Ptrs ps = p;
    ps.dST = nullptr; ps.dS0 = p.Rseg;
    scan_bwd_body<T, DK, DV, VAR, true, VBlock<T, DV, DK>::BV>(sm, H, ps, blockIdx.x);
}

// S_in(0) = the caller's initial state (or zero); S_in(g + 1) = M_g S_in(g) + N_g; the state after the last segment is
// the final state.  Backward (blockIdx.z = 1): D(G) = the caller's gradient with respect to the final state (or zero);
// every segment's end gradient dSout(g) = D(g + 1), D(g) = M_g^T D(g + 1) + R_g; D(0) is the gradient with respect to the
// initial state.  One workgroup per (chain, block of 32 state columns, direction): the columns evolve independently.
// fp32 on the matrix cores; the next segment's M and N (R) tile travel from global memory while the current product runs.
template <int DK, int DV> struct CombineSmem {
    static constexpr int LM = DK + 4, LSB = 32 + 4;
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
__global__ __launch_bounds__(NTHR) void k_seg_combine(CombineArgs a) {
    using SM = CombineSmem<DK, DV>;
    static_assert(DK % 32 == 0 && DK / 32 <= NTHR / 64, "one 32-row tile per wave");
    extern __shared__ __align__(16) unsigned char smem[];
    float *sM = reinterpret_cast<float *>(smem + SM::oM), *sS = reinterpret_cast<float *>(smem + SM::oS);
    const int chain = blockIdx.x, b = chain / a.H, h = chain - b * a.H, c0 = 32 * blockIdx.y;
    const bool bwd = (int)blockIdx.z + a.first_dir == 1;
    const int tid = threadIdx.x, wave = tid >> 6;
    const bool act = wave < DK / 32;
    const float *init = bwd ? a.dST : a.S0, *add = bwd ? a.Rseg : a.Nseg;
    float *start = bwd ? a.dSout : a.Sin, *last = bwd ? a.dS0 : a.ST;
    auto seg_of = [&](int i) __attribute__((always_inline)) { return ((long)(b * a.G + (bwd ? a.G - 1 - i : i)) * a.H + h); };
    TileRegs<float, DK, DK, NTHR> mreg;
    f32x16 nreg = zero16();
    auto request = [&](int i) __attribute__((always_inline)) { // M and the additive tile of step i, into registers
        const long seg = seg_of(i);
        mreg.load(a.Mseg + seg * DK * DK, DK, DK);
        if (act) acc_each(nreg, [&](int r, int c, float &val) { val = add[(seg * DK + 32 * wave + r) * DV + c0 + c]; });
    };
    request(0);
    for (int e = tid; e < DK * 32; e += NTHR) {
        const int i = e >> 5, j = e & 31;
        sS[i * SM::LSB + j] = init ? init[((long)chain * DK + i) * DV + c0 + j] : 0.f;
    }
    lds_barrier(); // (LDS only: the requests and stores in flight are not waited for)
    for (int i = 0; i < a.G; ++i) {
        const long seg = seg_of(i);
        for (int e = tid; e < DK * 32; e += NTHR) { // this segment starts from (backward: ends with) the current value
            const int r = e >> 5, j = e & 31;
            start[(seg * DK + r) * DV + c0 + j] = sS[r * SM::LSB + j];
        }
        mreg.store(sM, SM::LM);
        f32x16 acc = nreg;
        lds_barrier();
        if (i + 1 < a.G) request(i + 1);
        if (act) {
            if (bwd) mma<DK, true, true, float>(acc, sM + 32 * wave, SM::LM, sS, SM::LSB); // M^T D: down the rows of M
            else mma<DK, false, true, float>(acc, sM + 32 * wave * SM::LM, SM::LM, sS, SM::LSB);
        }
        lds_barrier(); // every wave has read the old value
        if (act) acc_to_lds<float>(sS, SM::LSB, 32 * wave, 0, acc);
        lds_barrier();
    }
    if (last)
        for (int e = tid; e < DK * 32; e += NTHR) {
            const int r = e >> 5, j = e & 31;
            last[((long)chain * DK + r) * DV + c0 + j] = sS[r * SM::LSB + j];
        }
}

// scan_bwd_body: reverse over chunks, carrying dS (gradient w.r.t. the chunk-initial state):
//   dUt = P^T dO + K dS';  dV = T^T dUt;  dS = dS' + Q^T dO - W^T dUt
// Per chunk it leaves dS'^T in the workspace (the transposed LDS copy, written out by the loader waves) and stores dV.
// In bf16 the product for dV reads dUt rounded, and the diagonal of T is beta (prologue variant: the fp32 sigmoid) rounded, one
// factor for a whole row.  The diagonal is the largest term of a row, so it is put in from the fp32 accumulators instead:
// dV = T^T bf16(dUt) + (beta dUt - bf16(beta) bf16(dUt)).  That brings dV 14 to 17 % closer to the exact one (rms, against 64
// bits) and makes up for the rounding that storing dV adds to dbeta, which the chunk kernel forms from it; it costs 2 to 4 %
// of the scan (16 384 tokens of width 2048: d = 64 118 -> 123 us, d = 256 229 -> 233).  The factors of dUt and bf16(dUt) come
// from two tables, and so a masked token (beta zero, or below kTinyBeta) costs nothing here: its row of T^T has nothing but the
// diagonal, beta, and with factors 1 and 0 the row that is stored is dUt_i, which the chunk kernel makes G_i and beta_i G_i from.
template <typename T, int DK, int DV, int BV> struct ScanBwdSmem {
    static constexpr int LQ = ldn<T>(DK), LK = ldn<T>(DK), LD = ldn<T>(BV), LS = ldc<T>(DK), LT = ldc<T>(C);
    static constexpr size_t oQ = 0;
    static constexpr size_t oK = oQ + align16(sizeof(T) * C * LQ);
    static constexpr size_t oW = oK + align16(sizeof(T) * C * LK);
    static constexpr size_t oDO = oW + align16(sizeof(T) * C * LQ);
    static constexpr size_t oDST = oDO + align16(sizeof(T) * C * LD);
    static constexpr size_t oDUT = oDST + align16(sizeof(T) * BV * LS);
    static constexpr size_t oT = oDUT + align16(sizeof(T) * BV * LT);
    static constexpr size_t szT = align16(sizeof(T) * C * LT);       // two T buffers, alternating by chunk parity
    // P^T; in the interval after its use, the staging tiles of the chain waves for dV
    static constexpr size_t oPT = oT + 2 * szT, oStage = oPT;
    static constexpr size_t szPT = cmax(szT, ScanMap<DK, BV>::U_TILES * sizeof(T) * Stage<T>::ELEMS);
    static constexpr size_t oGi = oPT + szPT;                        // gated: 1 / gamma_i, two tables, alternating as T
    static constexpr size_t oDiag = oGi + 2 * sizeof(float) * C;     // factors of dUt_i and of its rounded value in dV_i, two tables each
    static constexpr size_t bytes = oDiag + 4 * sizeof(float) * C;
};

// STATE = true: only the gradient with respect to the initial state leaves the kernel (the first pass of a backward
// pass that is split over segments of the sequence).
template <typename T, int DK, int DV, int VAR, bool STATE, int BV>
__device__ __forceinline__ void scan_bwd_body(const SeqMap &sm, int H, const Ptrs &p, int bid) {
    using SM = ScanBwdSmem<T, DK, DV, BV>;
    constexpr bool GATED = VAR == VAR_GATED, PRO = VAR == VAR_PROLOGUE; // (q and k are the mapped ones in every variant)
    constexpr int NV = DV / BV;
    using Map = ScanMap<DK, BV>;
    constexpr int NWT = (Map::W_TILES + 3) / 4; // W tiles per chain wave
    extern __shared__ __align__(16) unsigned char smem[];
    T *sQ = reinterpret_cast<T *>(smem + SM::oQ);
    T *sK = reinterpret_cast<T *>(smem + SM::oK);
    T *sW = reinterpret_cast<T *>(smem + SM::oW);
    T *sDO = reinterpret_cast<T *>(smem + SM::oDO);
    T *sDST = reinterpret_cast<T *>(smem + SM::oDST);
    T *sDUT = reinterpret_cast<T *>(smem + SM::oDUT);
    T *sT0 = reinterpret_cast<T *>(smem + SM::oT), *sT1 = reinterpret_cast<T *>(smem + SM::oT + SM::szT);
    T *sPT = reinterpret_cast<T *>(smem + SM::oPT);
    T *stg = reinterpret_cast<T *>(smem + SM::oStage) + ((threadIdx.x >> 6) % ScanMap<DK, BV>::U_TILES) * Stage<T>::ELEMS;
    float *sGi = reinterpret_cast<float *>(smem + SM::oGi), *sDiag = reinterpret_cast<float *>(smem + SM::oDiag);
    constexpr bool DIAG = !STATE && (sizeof(T) == 2 || !PRO); // a diagonal term of dV from the accumulators (fp32: the masked rows' only)
    constexpr bool kWholeLines = BV * sizeof(T) >= 128; // see scan_fwd_body
    constexpr bool gated = GATED; // compile-time, so the plain kernels carry none of the gate's registers
    // the gated kernels, and those with d_k = 256, request operand fragments in smaller batches: they have no registers to spare
    constexpr int MB = GATED ? 2 : (sizeof(T) == 4 ? 2 : (DK > 128 ? 4 : 0));

    int chain, vbi;
    if (!chain_of_block(bid, sm.N * H, NV, chain, vbi)) return;
    int n = chain / H;
    const int h = chain - n * H, vb = vbi * BV;
    if (sm.order) { n = sm.order[n]; chain = n * H + h; } // packed: longest sequences first
    const int wave = threadIdx.x >> 6;
    int t0, len, cb;
    sm.seq(n, t0, len, cb);
    const int nchunks = (len + C - 1) / C;
    const Map m(wave);
    const bool loader = wave >= 4;
    const int lt = threadIdx.x - NTL;
    // The dV tiles belong to the waves whose accumulators hold dUt; in fp32 to the two chain waves that own none (a product over
    // 64 is 32 dependent steps of 64 cycles there, and the owners have one in the same interval; the reverse scan of 3 x 1500
    // tokens, 8 heads of 64: 212 -> 170 us).
    static_assert(sizeof(T) == 2 || Map::U_TILES == 2, "fp32 column blocks are 32 wide");
    const int dvw = sizeof(T) == 2 ? wave : wave - 2, va = (dvw & 3) / Map::NVT, vb2 = (dvw & 3) % Map::NVT; // tile (va, vb2)
    const bool does_dv = !STATE && dvw >= 0 && dvw < Map::U_TILES;
    // waves 0..3 build the tiles (pmi, pni) = (0,0), (0,1), (1,1), (1,0) of P^T; the last one is all zero
    const int pmi = wave >> 1, pni = (wave == 1) | (wave == 2);

    f32x16 dS = zero16();
    if (m.has_s && p.dST) {
        const float *src = p.dST + (long)chain * DK * DV + vb;
        acc_each(dS, [&](int r, int c, float &val) { val = src[(long)(32 * m.sa + r) * DV + 32 * m.sb + c]; });
    }
    __builtin_amdgcn_s_waitcnt(0x0F70); // vmcnt(0): see k_scan_fwd

    struct Regs {
        TileRegs<T, C, DK, NTL> q, k;
        TileRegs<T, C, BV, NTL> d_o;
        TileRegs<T, C, C, NTL> t;
        float dos[TileRegs<T, C, BV, NTL>::NIT], gi; // gated: gamma of this lane's dO rows; one entry of the 1 / gamma table
        T beta;                                      // one row's beta (logit), in storage format (converting here would wait for the load)
    } r;
    auto fetch_a = [&](int ic) __attribute__((always_inline)) {
        const int nvalid = min(C, len - ic * C);
        const long row0 = (long)t0 + (long)ic * C;
        r.q.template load_aux<kAuxKeep>((const T *)p.q + (row0 * H + h) * DK, (long)H * DK, nvalid, lt);
        r.k.template load_aux<kAuxKeep>((const T *)p.k + (row0 * H + h) * DK, (long)H * DK, nvalid, lt);
    };
    auto fetch_b = [&](int ic) __attribute__((always_inline)) {
        const int nvalid = min(C, len - ic * C);
        const long row0 = (long)t0 + (long)ic * C;
        const long tile = ((long)(cb + ic) * H + h);
        r.d_o.template load_aux<kAuxKeep>((const T *)p.d_o + (row0 * H + h) * DV + vb, (long)H * DV, nvalid, lt);
        r.t.template load_aux<kAuxKeep>((const T *)p.Tm + tile * C * C, C, C, lt);
        if (gated) {
            r.d_o.load_row_factors(r.dos, p.gam + tile * 2 * C, lt);
            if (lt < C) r.gi = p.gam[tile * 2 * C + C + lt];
        }
        if (DIAG && lt < C) r.beta = ((const T *)p.beta)[(row0 + min(lt, nvalid - 1)) * H + h]; // (dUt of a row past the end meets rows of zeros)
    };
    // As in the forward scan, the loader waves issue the global traffic of a step in one burst after
    // its first barrier: next chunk's loads, this chunk's dS'^T.
    auto stash = [&](int par) __attribute__((always_inline)) { // fetched tiles of a chunk of parity `par`: registers -> LDS
        r.q.store(sQ, SM::LQ, lt); r.k.store(sK, SM::LK, lt);
        if (gated) r.d_o.scale_rows(r.dos); // o_i = gamma_i o~_i, so the plain rule's output gradient is gamma_i dO_i
        r.d_o.store(sDO, SM::LD, lt);
        r.t.store(par ? sT1 : sT0, SM::LT, lt);
        if (gated && lt < C) sGi[par * C + lt] = r.gi;
        if (DIAG && lt < C) {
            const float bt = PRO ? sigmoid_f32(to_f32(r.beta)) : to_f32(r.beta);
            const bool tiny = !PRO && fabsf(bt) < kTinyBeta;
            sDiag[2 * par * C + lt] = tiny ? 1.f : sizeof(T) == 2 ? bt : 0.f;
            sDiag[(2 * par + 1) * C + lt] = tiny || sizeof(T) == 4 ? 0.f : -to_f32(from_f32<T>(bt));
        }
    };
    if (loader && nchunks > 0) { fetch_a(nchunks - 1); fetch_b(nchunks - 1); stash((nchunks - 1) & 1); }
    // gated: the state after the chunk is gamma_C times the plain rule's, so its gradient is scaled by
    // gamma_C on entry; every wave requests the value for the next step one step ahead
    float gCn = 1.f, gHere = 1.f; // gHere: gamma_C of the chunk of the current step
    if (gated && nchunks > 0) gCn = gHere = p.gam[((long)(cb + nchunks - 1) * H + h) * 2 * C + C - 1];
    // dS' of the last chunk (the gradient with respect to the state after it) goes to LDS here; every later one at the end
    // of the step that produced it: that interval reads only W and dUt^T, so the state gradient's LDS copy and the next
    // chunk's tiles can be written in it, and a chunk step takes three barrier intervals.
    if (gated) dS *= gCn;
    if (m.has_s && nchunks > 0) acc_to_lds_t<T>(sDST, SM::LS, 32 * m.sa, 32 * m.sb, dS);
    for (int ic = nchunks - 1; ic >= 0; --ic) {
        const long tile = ((long)(cb + ic) * H + h);
        const T *sT = (ic & 1) ? sT1 : sT0;
        if (gated && ic > 0) gCn = p.gam[(tile - H) * 2 * C + C - 1]; // for the end of this step
        lds_barrier();
        if (loader && ic > 0) fetch_a(ic - 1);
        // dS'^T to the workspace, in the interval whose length the chain waves' products set
        if (loader && !STATE) copy_out<T, BV, DK, NTL, true>((T *)p.dSc + (tile * DV + vb) * DK, sDST, SM::LS, lt);
        f32x16 acc = zero16();
        if (!loader) { // straight-line, as in the forward scan; the loader waves are busy with global memory meanwhile
            // (with more than two W tiles per wave, d_k = 256, the tiles are finished one at a time, as in the forward scan)
            constexpr bool SEQ = GATED || NWT > 2;
            f32x16 pa = zero16(); // P^T = triu(K Q^T), the transposed causal scores, computed as the tile (pni, pmi) of P
            mma<DK, false, false, T, SEQ, MB>(pa, sQ + 32 * pni * SM::LQ, SM::LQ, sK + 32 * pmi * SM::LK, SM::LK);
            if (m.does_u) // K dS' part of the dUt tile (ua, ub)
                mma<DK, false, false, T, SEQ, MB>(acc, sK + 32 * m.ua * SM::LK, SM::LK, sDST + 32 * m.ub * SM::LS, SM::LS);
            f32x16 w[NWT];
#pragma unroll
            for (int i = 0; i < NWT; ++i) { // W = T K (Eq. 11), computed as W^T = K^T T^T
                const int t = wave + 4 * i, wk = t % Map::NKT, wi = t / Map::NKT;
                w[i] = zero16();
                if (Map::W_TILES % 4 == 0 || t < Map::W_TILES) {
                    mma<C, true, false, T, SEQ, MB>(w[i], sK + 32 * wk, SM::LK, sT + 32 * wi * SM::LT, SM::LT);
                    if (NWT > 2) acc_to_lds_t<T>(sW, SM::LQ, 32 * wk, 32 * wi, w[i]);
                }
            }
            acc_each(pa, [&](int r, int c, float &val) { if (32 * pni + r < 32 * pmi + c) val = 0.f; });
            acc_to_lds_t<T>(sPT, SM::LT, 32 * pni, 32 * pmi, pa);
            if (NWT <= 2) {
#pragma unroll
                for (int i = 0; i < NWT; ++i) {
                    const int t = wave + 4 * i, wk = t % Map::NKT, wi = t / Map::NKT;
                    if (Map::W_TILES % 4 == 0 || t < Map::W_TILES) acc_to_lds_t<T>(sW, SM::LQ, 32 * wk, 32 * wi, w[i]);
                }
            }
        }
        lds_barrier();
        if (loader) {
            if (ic > 0) fetch_b(ic - 1);
        }
        if (m.does_u) { // + P^T dO; P^T is upper triangular
            if (m.ua == 0) mma<C, false, true, T, true, MB>(acc, sPT, SM::LT, sDO + 32 * m.ub, SM::LD);
            else mma<32, false, true, T, true, MB>(acc, sPT + 32 * SM::LT + 32, SM::LT, sDO + 32 * SM::LD + 32 * m.ub, SM::LD);
            acc_to_lds_t<T>(sDUT, SM::LT, 32 * m.ua, 32 * m.ub, acc);
        }
        if (m.has_s) mma<C, true, true, T, true, MB>(dS, sQ + 32 * m.sa, SM::LQ, sDO + 32 * m.sb, SM::LD); // + Q^T dO
        lds_barrier();
        if (m.has_s) { // - W^T dUt
            f32x16 wd = zero16();
            mma<C, true, false, T, true, MB>(wd, sW + 32 * m.sa, SM::LQ, sDUT + 32 * m.sb * SM::LT, SM::LT);
            dS -= wd;
        }
        if (ic > 0) {
            if (gated) { // across the boundary: out of this chunk's coordinates, into those of the chunk before
                dS *= gHere; // (one factor at a time: their product may leave the fp32 range)
                dS *= gCn;
                gHere = gCn;
            }
            if (m.has_s) acc_to_lds_t<T>(sDST, SM::LS, 32 * m.sa, 32 * m.sb, dS); // dS' of the next step
            if (loader) stash((ic - 1) & 1); // see k_scan_fwd
        }
        // dV = T^T dUt (T^T is upper triangular), formed and sent by the chain waves: the loader waves have the next chunk's
        // tiles to move in this interval
        if (does_dv) {
            f32x16 dv = zero16();
            int tx = threadIdx.x;
            if (sizeof(T) == 4) asm volatile("" : "+v"(tx)); // (its addresses are formed here, not carried through the loop: no registers to spare)
            if (va == 0) mma<C, true, false, T, true, MB>(dv, sT, SM::LT, sDUT + 32 * vb2 * SM::LT, SM::LT, tx);
            else mma<32, true, false, T, true, MB>(dv, sT + 32 * SM::LT + 32, SM::LT, sDUT + 32 * vb2 * SM::LT + 32, SM::LT, tx);
            if (DIAG && (sizeof(T) == 2 || __ballot(sDiag[2 * (ic & 1) * C + (tx & 63)] != 0.f))) { // (fp32: without a masked token there is no term)
                const int hh = (tx & 63) >> 5;
                const float *fa = sDiag + 2 * (ic & 1) * C + 32 * va + 4 * hh, *fr = fa + C;
#pragma unroll
                for (int e = 0; e < 16; ++e) {
                    const int r8 = 8 * (e >> 2) + (e & 3);
                    if constexpr (sizeof(T) == 2) dv[e] += fa[r8] * acc[e] + fr[r8] * to_f32(from_f32<T>(acc[e]));
                    else dv[e] += fa[r8] * sDUT[(32 * vb2 + (tx & 31)) * SM::LT + 32 * va + 4 * hh + r8]; // (nothing is rounded on the way to LDS)
                }
            }
            if (gated) acc_each(dv, [&](int rr, int, float &val) { val *= sGi[(ic & 1) * C + 32 * va + rr]; }, tx); // v_i = gamma_i v~_i
            acc_store<T, kWholeLines>(stg, (T *)p.dv + (((long)t0 + (long)ic * C) * H + h) * DV + vb, (long)H * DV, 32 * va, 32 * vb2, min(C, len - ic * C), dv, tx);
        }
    }
    if (p.dS0 && m.has_s) {
        float *dst = p.dS0 + (long)chain * DK * DV + vb;
        if (gated) dS *= gHere; // out of the first chunk's coordinates
        acc_each(dS, [&](int r, int c, float &val) { dst[(long)(32 * m.sa + r) * DV + 32 * m.sb + c] = val; });
    }
}

// The backward pass's two scans in one launch.  They do not depend on each other (the recompute
// scan needs T; the reverse scan needs T and P^T), so the first half of the grid runs the reverse
// scan and the second half the recompute scan: a CU picks up one of each with no kernel boundary
// in between.  `half` = workgroups per scan.
template <typename T, int DK, int DV, int VAR, int BV>
__global__ __launch_bounds__(NTS) void k_scan_pair(SeqMap sm, int H, Ptrs p, int half) {
    if ((int)blockIdx.x < half) scan_bwd_body<T, DK, DV, VAR, false, BV>(sm, H, p, blockIdx.x);
    else scan_fwd_body<T, DK, DV, SCAN_STORE, VAR == VAR_PROLOGUE ? VAR_PLAIN : VAR, BV>(sm, H, p, blockIdx.x - half);
}
// the reverse scan alone, for a backward pass that finds the forward scan's tiles already in the workspace
template <typename T, int DK, int DV, int VAR, int BV>
__global__ __launch_bounds__(NTS) void k_scan_bwd(SeqMap sm, int H, Ptrs p) {
    scan_bwd_body<T, DK, DV, VAR, false, BV>(sm, H, p, blockIdx.x);
}

// =============================================================================================
// The chunk-parallel backward kernel (dn_chunk_local.hpp).  Workgroups are persistent: each walks over
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
