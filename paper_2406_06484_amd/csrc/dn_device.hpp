// Device-side building blocks for the gfx950 DeltaNet kernels: MFMA tile products from LDS,
// accumulator <-> LDS/global movers, tile loaders, the 64x64 unit-lower-triangular inverse.
// The chunk is C = 64 tokens; the prep kernel runs 4 wavefronts, the chunk kernel 8, the scans 5 to 12.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace dn {

constexpr int C = 64;     // chunk size (section 3.2)
constexpr int NTHR = 256; // threads per workgroup
constexpr int NWAVE = 4;

typedef __bf16 bf16;
typedef bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

// Workgroup barrier that orders LDS traffic only.  __syncthreads() also drains every outstanding
// global load and store of the wave (it is a full workgroup fence), which would serialise the
// register prefetch of the next chunk and the output stores with the barrier.  Every barrier in
// these kernels guards LDS contents only; nothing written to global memory is read back by the
// same launch.
__device__ inline void lds_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

// Global loads go through raw buffer descriptors: one 32-bit per-lane offset serves a whole tile
// (the row step rides in the scalar offset), and rows past the end of a ragged chunk are masked by
// pointing their lanes beyond the descriptor's range, which makes the hardware return zeros.
// This keeps 64-bit per-load address pairs and exec-mask branches out of the prefetch code.
typedef int i32x4 __attribute__((ext_vector_type(4)));
// Cache-policy bits of the loads and stores, per stream of tiles (0 = default, 2 = non-temporal; measured variant by
// variant on the fwd+bwd step, kernels of one step timed side by side on the same device):
//   tiles the launch reads once and no later kernel of the same call needs: non-temporal loads (every operand of the
//     chunk kernel; V in the forward scan, whose two workgroups per chain read different column blocks)
//   tiles that the other workgroup of the chain reads too (Q, K, T in the scans) or that the next kernel of the call reads
//     (K in k_wy_prep, dO in the reverse scan): default policy, they are found in the L2 or the memory-side cache
//   every tile store of the scans, k_wy_prep and the chunk kernel: non-temporal (nothing is read back by the same launch)
constexpr int kAuxOnce = 2, kAuxKeep = 0;
constexpr int kBufRange = 0x40000000; // bytes covered by a descriptor; offsets >= this read as zero
__device__ inline __amdgpu_buffer_rsrc_t make_rsrc(const void *base, int range = kBufRange) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(base), 0, range, 0x00020000);
}
// AUX = the instruction's cache-policy bits: 0 = default, 2 = non-temporal (data that this launch reads once)
template <int AUX = 0> __device__ inline uint4 buf_load16(__amdgpu_buffer_rsrc_t rs, int voff, int soff) {
    return __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(rs, voff, soff, AUX));
}

// Per-element-type constants: LDS row padding (elements) and elements per 16 bytes.
template <typename T> struct El;
template <> struct El<float> { static constexpr int PAD = 4; static constexpr int VEC = 4; };
template <> struct El<bf16>  { static constexpr int PAD = 16; static constexpr int VEC = 8; };

template <typename T> __host__ __device__ constexpr int ldn(int cols) { return cols + El<T>::PAD; }
// leading dimension for tiles that are only ever read with the contraction index contiguous
template <typename T> __host__ __device__ constexpr int ldc(int cols) { return cols + 16 / (int)sizeof(T); }

__device__ inline float to_f32(float x) { return x; }
__device__ inline float to_f32(bf16 x) { return (float)x; }
template <typename T> __device__ inline T from_f32(float x) { return (T)x; }
// logistic function in explicit single-rounding steps, so that every kernel that evaluates it gets the same bits
__device__ inline float sigmoid_f32(float x) { return __frcp_rn(__fadd_rn(1.f, __expf(-x))); }
// ... and with the hardware reciprocal (1 ulp), for values that no other kernel has to reproduce bit for bit
__device__ inline float sigmoid_fast_f32(float x) { return __builtin_amdgcn_rcpf(1.f + __expf(-x)); }

// Where the chains live.  Dense batches are N = B sequences of length L at rows n*L; packed
// batches read cu_seqlens and a device-computed prefix of per-sequence chunk counts.
struct SeqMap {
    const int32_t *cu;   // device [N+1] or nullptr
    const int32_t *coff; // device [N+1] chunk offsets (packed only)
    const int32_t *order; // device [N] sequences by decreasing length (packed only), for the chain-serial kernels
    int N, L, ncd;       // ncd = chunks per dense sequence
    __device__ void seq(int n, int &t0, int &len, int &cb) const {
        if (cu) { t0 = cu[n]; len = cu[n + 1] - t0; cb = coff[n]; }
        else { t0 = n * L; len = L; cb = n * ncd; }
    }
    // maps a global chunk id to (sequence, chunk within it); false if past the end
    __device__ bool chunk(int gid, int &n, int &ic) const {
        if (!cu) {
            if (gid >= N * ncd) return false;
            n = gid / ncd; ic = gid - n * ncd; return true;
        }
        if (gid >= coff[N]) return false;
        int lo = 0, hi = N; // coff[lo] <= gid < coff[hi]
        while (hi - lo > 1) { int mid = (lo + hi) >> 1; if (coff[mid] <= gid) lo = mid; else hi = mid; }
        n = lo; ic = gid - coff[lo]; return true;
    }
};

// ---------------------------------------------------------------------------------------------
// The 32x32 MFMAs.  v_mfma_f32_32x32x16_bf16: lane l feeds row/col (l & 31) and 8 consecutive k
// starting at 8*(l >> 5); v_mfma_f32_32x32x2_f32: one k = (l >> 5).  The accumulator holds, for
// lane l, column (l & 31) and rows 8*g + 4*(l >> 5) + i at index 4*g + i.
//
// Operand fragments for the 32x32 MFMAs, from LDS, in two storage orders:
//   KC  storage [n][k], contraction index contiguous  (one 16-byte read per lane in bf16)
//   KS  storage [k][n], contraction index strided     (bf16: two ds_read_b64_tr_b16, the CDNA4
//       transposing LDS read; fp32: a plain read, since an fp32 fragment is one element per lane)
// `base` points at (n0, k = 0) for KC and at (k = 0, n0) for KS.  Both orders give lane l the
// operand row/column n0 + (l & 31) and, in bf16, k = k0 + 8*(l >> 5) + 0..7.
typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef short s16x8 __attribute__((ext_vector_type(8)));

// (`tx`: the thread index as the caller wants it seen.  The default is threadIdx.x itself; a kernel that wants the per-lane
// address arithmetic formed where it is used, rather than hoisted out of its outer loop and carried through it, passes a
// copy it has taken through an empty asm.)
__device__ inline bf16x8 frag_kc(const bf16 *base, int ld, int k0, int tx = threadIdx.x) {
    const int lane = tx & 63;
    return *reinterpret_cast<const bf16x8 *>(base + (lane & 31) * ld + k0 + 8 * (lane >> 5));
}
__device__ inline bf16x8 frag_ks(const bf16 *base, int ld, int k0, int tx = threadIdx.x) {
    // Within each group of 16 lanes the transposing read hands lane i the 16-bit element (i & 3) of
    // the four 8-byte rows addressed by lanes (i >> 2), (i >> 2) + 4, + 8, + 12.  With lane i
    // pointing at row k0' + (i >> 2), columns 4*(i & 3).., lane i ends up with column i, rows k0'..k0'+3.
    const int lane = tx & 63, i = lane & 15;
    const bf16 *p = base + (k0 + 8 * (lane >> 5) + (i >> 2)) * ld + (lane & 16) + 4 * (i & 3);
    typedef __attribute__((address_space(3))) s16x4 lds_s16x4;
    const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4 *)(p));
    const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4 *)(p + 4 * ld));
    const s16x8 v = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
    return __builtin_bit_cast(bf16x8, v);
}
__device__ inline float frag_kc(const float *base, int ld, int k0, int tx = threadIdx.x) {
    const int lane = tx & 63;
    return base[(lane & 31) * ld + k0 + (lane >> 5)];
}
__device__ inline float frag_ks(const float *base, int ld, int k0, int tx = threadIdx.x) {
    const int lane = tx & 63;
    return base[(k0 + (lane >> 5)) * ld + (lane & 31)];
}
__device__ inline void mfma32(f32x16 &acc, bf16x8 a, bf16x8 b) { acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, acc, 0, 0, 0); }
__device__ inline void mfma32(f32x16 &acc, float a, float b) { acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a, b, acc, 0, 0, 0); }
template <typename T> struct FragOf;
template <> struct FragOf<bf16> { typedef bf16x8 type; static constexpr int KPL = 8; };
template <> struct FragOf<float> { typedef float type; static constexpr int KPL = 1; };
template <typename T> struct KStep;
template <> struct KStep<bf16> { static constexpr int value = 16; };
template <> struct KStep<float> { static constexpr int value = 2; };

// acc(32x32) += A * B over KDIM contraction steps; AKS / BKS select the storage order of each operand.
// The operand fragments of up to BATCH steps are requested from LDS before the first MFMA of the
// batch issues (and the next batch's before this batch's MFMAs), so one LDS latency is exposed per
// product instead of one per pair of steps, which is what the compiler's own schedule gives.
template <typename T> struct MmaBatch;
template <> struct MmaBatch<bf16> { static constexpr int value = 8; };   // 8 steps x 2 operands x 4 VGPRs
template <> struct MmaBatch<float> { static constexpr int value = 16; }; // 16 steps x 2 operands x 1 VGPR
template <int KDIM, bool AKS, bool BKS, typename T, bool FENCE = true, int BATCH_ = 0>
__device__ inline void mma(f32x16 &acc, const T *A, int lda, const T *B, int ldb, int tx = threadIdx.x) {
    constexpr int KS = KStep<T>::value, N = KDIM / KS;
    constexpr int WANT = BATCH_ ? BATCH_ : MmaBatch<T>::value;
    constexpr int BATCH = N < WANT ? N : WANT, NB = (N + BATCH - 1) / BATCH;
    static_assert(N % BATCH == 0, "contraction length must be a multiple of the batch");
    typedef typename FragOf<T>::type frag_t;
    frag_t a[2][BATCH], b[2][BATCH];
#pragma unroll
    for (int j = 0; j < BATCH; ++j) {
        a[0][j] = AKS ? frag_ks(A, lda, j * KS, tx) : frag_kc(A, lda, j * KS, tx);
        b[0][j] = BKS ? frag_ks(B, ldb, j * KS, tx) : frag_kc(B, ldb, j * KS, tx);
    }
#pragma unroll
    for (int ib = 0; ib < NB; ++ib) {
        if (ib + 1 < NB) {
#pragma unroll
            for (int j = 0; j < BATCH; ++j) {
                const int k0 = ((ib + 1) * BATCH + j) * KS;
                a[(ib + 1) & 1][j] = AKS ? frag_ks(A, lda, k0, tx) : frag_kc(A, lda, k0, tx);
                b[(ib + 1) & 1][j] = BKS ? frag_ks(B, ldb, k0, tx) : frag_kc(B, ldb, k0, tx);
            }
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int j = 0; j < BATCH; ++j) mfma32(acc, a[ib & 1][j], b[ib & 1][j]);
    }
    // FENCE keeps the scheduler from hoisting the next product's operand loads over this one (register
    // pressure); without it the next product's loads may overlap this product's MFMAs.
    if (FENCE) __builtin_amdgcn_sched_barrier(0);
}

// Two products with the same B operand: acc1 += A1 * B, acc2 += A2 * B; B's fragments are read from LDS once.
template <int KDIM, bool A1KS, bool A2KS, bool BKS, typename T, int BATCH_>
__device__ inline void mma_shared_b(f32x16 &acc1, f32x16 &acc2, const T *A1, int lda1, const T *A2, int lda2, const T *B, int ldb,
                                    int tx = threadIdx.x) {
    constexpr int KS = KStep<T>::value, N = KDIM / KS;
    constexpr int BATCH = N < BATCH_ ? N : BATCH_, NB = N / BATCH;
    static_assert(N % BATCH == 0, "contraction length must be a multiple of the batch");
    typedef typename FragOf<T>::type frag_t;
    frag_t a1[2][BATCH], a2[2][BATCH], b[2][BATCH];
#pragma unroll
    for (int j = 0; j < BATCH; ++j) {
        b[0][j] = BKS ? frag_ks(B, ldb, j * KS, tx) : frag_kc(B, ldb, j * KS, tx);
        a1[0][j] = A1KS ? frag_ks(A1, lda1, j * KS, tx) : frag_kc(A1, lda1, j * KS, tx);
        a2[0][j] = A2KS ? frag_ks(A2, lda2, j * KS, tx) : frag_kc(A2, lda2, j * KS, tx);
    }
#pragma unroll
    for (int ib = 0; ib < NB; ++ib) {
        if (ib + 1 < NB) {
#pragma unroll
            for (int j = 0; j < BATCH; ++j) {
                const int k0 = ((ib + 1) * BATCH + j) * KS;
                b[(ib + 1) & 1][j] = BKS ? frag_ks(B, ldb, k0, tx) : frag_kc(B, ldb, k0, tx);
                a1[(ib + 1) & 1][j] = A1KS ? frag_ks(A1, lda1, k0, tx) : frag_kc(A1, lda1, k0, tx);
                a2[(ib + 1) & 1][j] = A2KS ? frag_ks(A2, lda2, k0, tx) : frag_kc(A2, lda2, k0, tx);
            }
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int j = 0; j < BATCH; ++j) {
            mfma32(acc1, a1[ib & 1][j], b[ib & 1][j]);
            mfma32(acc2, a2[ib & 1][j], b[ib & 1][j]);
        }
    }
    __builtin_amdgcn_sched_barrier(0);
}

__device__ inline f32x16 zero16() {
    f32x16 z;
#pragma unroll
    for (int i = 0; i < 16; ++i) z[i] = 0.f;
    return z;
}

// visit every accumulator element: f(row, col, value&) with row, col inside the 32x32 tile
template <typename F> __device__ inline void acc_each(f32x16 &acc, F f, int tx = threadIdx.x) {
    const int lane = tx & 63, col = lane & 31, h = lane >> 5;
#pragma unroll
    for (int g = 0; g < 4; ++g)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            float v = acc[4 * g + i]; // vector elements cannot bind to a reference
            f(8 * g + 4 * h + i, col, v);
            acc[4 * g + i] = v;
        }
}
// visit runs of 4 consecutive rows: f(row0, col, v0, v1, v2, v3)
template <typename F> __device__ inline void acc_each4(const f32x16 &acc, F f, int tx = threadIdx.x) {
    const int lane = tx & 63, col = lane & 31, h = lane >> 5;
#pragma unroll
    for (int g = 0; g < 4; ++g) f(8 * g + 4 * h, col, acc[4 * g], acc[4 * g + 1], acc[4 * g + 2], acc[4 * g + 3]);
}

// Lane exchanges inside a row of 16 lanes on the vector ALU (a __shfl_xor goes through the LDS).  The distances 8, 4, 2, 1 pair
// lane l with l ^ 8, l ^ 7 (the mirror image within 8), l ^ 2 and l ^ 1: a chain of sums in that order, or in the reverse one
// from any of them, covers the same lanes as the butterfly.
template <int D> __device__ inline float lane_across(float x) {
    constexpr int ctrl = D == 8 ? 0x128 /* row_ror:8 */ : D == 4 ? 0x141 /* row_half_mirror */ : D == 2 ? 0x4e /* quad_perm 2,3,0,1 */ : 0xb1 /* quad_perm 1,0,3,2 */;
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), ctrl, 0xf, 0xf, false));
}
// sum over N neighbouring lanes (N = 4, 8, 16), delivered to all of them
template <int N> __device__ inline float lane_sum(float x) {
    static_assert(N == 4 || N == 8 || N == 16, "inside a row of lanes");
    x += lane_across<1>(x);
    x += lane_across<2>(x);
    if (N >= 8) x += lane_across<4>(x);
    if (N >= 16) x += lane_across<8>(x);
    return x;
}
// dst[r] = sum over the columns of row r of the 32 x 32 tile.  Each of the first four steps sends one half of the remaining rows
// to the lane across and keeps the other, so a tile takes 16 exchanges instead of 80; the order of the additions is fixed.
template <int D> __device__ inline void row_sums_step(float (&v)[16], int lane) {
    const bool hi = (lane & D) != 0;
#pragma unroll
    for (int e = 0; e < D; ++e) {
        const float send = hi ? v[e] : v[e + D], keep = hi ? v[e + D] : v[e];
        v[e] = keep + lane_across<D>(send);
    }
}
__device__ inline void row_sums(float *dst, const f32x16 &acc, int tx = threadIdx.x) {
    const int lane = tx & 63;
    float v[16];
#pragma unroll
    for (int e = 0; e < 16; ++e) v[e] = acc[e];
    row_sums_step<8>(v, lane);
    row_sums_step<4>(v, lane);
    row_sums_step<2>(v, lane);
    row_sums_step<1>(v, lane);
    v[0] += __shfl_xor(v[0], 16); // lane & 15 is the element index now
    if (!(lane & 16)) dst[8 * ((lane & 15) >> 2) + 4 * (lane >> 5) + (lane & 3)] = v[0];
}

__device__ inline void st4(float *p, float a, float b, float c, float d) {
    *reinterpret_cast<f32x4 *>(p) = f32x4{a, b, c, d};
}
__device__ inline void st4(bf16 *p, float a, float b, float c, float d) {
    *reinterpret_cast<bf16x4 *>(p) = bf16x4{(bf16)a, (bf16)b, (bf16)c, (bf16)d};
}

// four neighbouring elements, from or to LDS or global memory (16 bytes, 8 in bf16)
template <typename T> __device__ inline void ld4(T (&x)[4], const T *p) {
    struct alignas(4 * sizeof(T)) quad { T e[4]; };
    const quad q = *reinterpret_cast<const quad *>(p);
#pragma unroll
    for (int i = 0; i < 4; ++i) x[i] = q.e[i];
}
template <typename T> __device__ inline void st4v(T *p, const T (&x)[4]) {
    struct alignas(4 * sizeof(T)) quad { T e[4]; };
    *reinterpret_cast<quad *>(p) = quad{{x[0], x[1], x[2], x[3]}};
}
// tile (32x32) of the accumulator -> LDS, row-major destination dst[row][col]
template <typename T> __device__ inline void acc_to_lds(T *dst, int ld, int row0, int col0, f32x16 &acc, int tx = threadIdx.x) {
    acc_each(acc, [&](int r, int c, float &v) { dst[(row0 + r) * ld + col0 + c] = from_f32<T>(v); }, tx);
}
// ... and transposed: dstT[col][row], 4 consecutive rows per store
template <typename T> __device__ inline void acc_to_lds_t(T *dstT, int ldT, int row0, int col0, const f32x16 &acc, int tx = threadIdx.x) {
    acc_each4(acc, [&](int r, int c, float a, float b, float cc, float d) {
        st4(dstT + (col0 + c) * ldT + row0 + r, a, b, cc, d);
    }, tx);
}
// Wave-private LDS staging for coalesced tile stores.  A 32 x 32 accumulator tile is first laid
// out row-major in LDS (cheap narrow LDS writes), then each lane moves 16 bytes at a time to global
// memory, so a store instruction covers whole 64-byte (bf16) or 128-byte (fp32) row segments.
// Scattered 2-byte global stores straight from the accumulator layout cost ~100 cycles apiece.
template <typename T> struct Stage {
    static constexpr int LD = 32 + 16 / (int)sizeof(T);       // row stride in elements, 16-byte aligned
    static constexpr int ELEMS = 32 * LD;                      // per wave
    static constexpr int SEGS = 32 * (int)sizeof(T) / 16;      // 16-byte segments per row
};
__device__ inline void wave_lds_fence() { asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory"); }

// ONCE: non-temporal store, for output that nothing reads again before the launch ends
typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
template <typename T, bool ONCE = false>
__device__ inline void stage_flush(const T *stage, T *dst, long row_stride, int row0, int col0, int nvalid, int tx = threadIdx.x) {
    const int lane = tx & 63;
    wave_lds_fence();
#pragma unroll
    for (int it = 0; it < 32 * Stage<T>::SEGS / 64; ++it) {
        const int idx = it * 64 + lane, r = idx / Stage<T>::SEGS, sg = idx % Stage<T>::SEGS;
        if (row0 + r < nvalid) {
            const u32x4 val = *reinterpret_cast<const u32x4 *>(stage + r * Stage<T>::LD + sg * El<T>::VEC);
            u32x4 *to = reinterpret_cast<u32x4 *>(dst + (long)(row0 + r) * row_stride + col0 + sg * El<T>::VEC);
            if (ONCE) __builtin_nontemporal_store(val, to);
            else *to = val;
        }
    }
    wave_lds_fence(); // the staging tile may be rewritten right away
}
// stage_flush that also returns row dot products of the staged tile with the matching 32 x 32 block of
// an LDS-resident matrix `other` (leading dimension ldo): slot[row0 + r] = sum_c stage(r, c) *
// other(row0 + r, col0 + c), written by one lane per row.  Used for the per-token terms of the gate gradient.
template <typename T>
__device__ inline void stage_flush_dot(const T *stage, T *dst, long row_stride, int row0, int col0, int nvalid,
                                       const T *other, int ldo, float *slot) {
    constexpr int SEGS = Stage<T>::SEGS, VEC = El<T>::VEC;
    const int lane = threadIdx.x & 63;
    wave_lds_fence();
#pragma unroll
    for (int it = 0; it < 32 * SEGS / 64; ++it) {
        const int idx = it * 64 + lane, r = idx / SEGS, sg = idx % SEGS;
        alignas(16) T a[VEC], b[VEC];
        *reinterpret_cast<uint4 *>(a) = *reinterpret_cast<const uint4 *>(stage + r * Stage<T>::LD + sg * VEC);
        *reinterpret_cast<uint4 *>(b) = *reinterpret_cast<const uint4 *>(other + (row0 + r) * ldo + col0 + sg * VEC);
        if (row0 + r < nvalid)
            *reinterpret_cast<uint4 *>(dst + (long)(row0 + r) * row_stride + col0 + sg * VEC) = *reinterpret_cast<const uint4 *>(a);
        float s = 0.f;
#pragma unroll
        for (int u = 0; u < VEC; ++u) s += to_f32(a[u]) * to_f32(b[u]);
#pragma unroll
        for (int d = 1; d < SEGS; d <<= 1) s += __shfl_xor(s, d); // the SEGS lanes of one row are adjacent
        if (sg == 0) slot[row0 + r] = s;
    }
    wave_lds_fence();
}
// dst[row0 + r][col0 + c] = acc(r, c), rows >= nvalid dropped; `stage` is this wave's staging tile
template <typename T, bool ONCE = false>
__device__ inline void acc_store(T *stage, T *dst, long row_stride, int row0, int col0, int nvalid, f32x16 &acc, int tx = threadIdx.x) {
    acc_to_lds<T>(stage, Stage<T>::LD, 0, 0, acc, tx);
    stage_flush<T, ONCE>(stage, dst, row_stride, row0, col0, nvalid, tx);
}
// ---------------------------------------------------------------------------------------------
// A ROWS x COLS tile fetched from global memory into registers (16 bytes per lane and step; rows >=
// nvalid read as zero), to be parked while LDS is busy and stored to LDS later.
template <typename T, int ROWS, int COLS, int NT = NTHR> struct TileRegs {
    static constexpr int VEC = El<T>::VEC, TPR = COLS / VEC, RPI = NT / TPR, NIT = ROWS / RPI;
    static_assert(COLS % VEC == 0 && NT % TPR == 0 && ROWS % RPI == 0, "tile shape");
    uint4 v[NIT];
    // `t` is the caller's index among the NT threads that share the tile (defaults to the whole workgroup)
    template <int AUX> __device__ inline void load_aux(const T *src, long row_stride, int nvalid, int t) {
        const int tr = t / TPR, tc = (t % TPR) * VEC;
        const __amdgpu_buffer_rsrc_t rs = make_rsrc(src);
        const int rs_bytes = (int)row_stride * (int)sizeof(T);
        const int voff = tr * rs_bytes + tc * (int)sizeof(T);
#pragma unroll
        for (int it = 0; it < NIT; ++it)
            v[it] = buf_load16<AUX>(rs, it * RPI + tr < nvalid ? voff : kBufRange, it * RPI * rs_bytes);
    }
    __device__ inline void load(const T *src, long row_stride, int nvalid, int t = threadIdx.x) { load_aux<0>(src, row_stride, nvalid, t); }
    // for a tile that no other workgroup of the launch reads: non-temporal, it does not displace what the caches hold
    __device__ inline void load_once(const T *src, long row_stride, int nvalid, int t = threadIdx.x) { load_aux<kAuxOnce>(src, row_stride, nvalid, t); }
    __device__ inline void store(T *dst, int ld, int t = threadIdx.x) const {
        const int tr = t / TPR, tc = (t % TPR) * VEC;
#pragma unroll
        for (int it = 0; it < NIT; ++it) *reinterpret_cast<uint4 *>(dst + (it * RPI + tr) * ld + tc) = v[it];
    }
    // ... with the sign of every element flipped (exact)
    __device__ inline void store_neg(T *dst, int ld, int t = threadIdx.x) const {
        constexpr unsigned S = sizeof(T) == 2 ? 0x80008000u : 0x80000000u;
        const int tr = t / TPR, tc = (t % TPR) * VEC;
#pragma unroll
        for (int it = 0; it < NIT; ++it)
            *reinterpret_cast<uint4 *>(dst + (it * RPI + tr) * ld + tc) = make_uint4(v[it].x ^ S, v[it].y ^ S, v[it].z ^ S, v[it].w ^ S);
    }
    // sum over the elements this lane holds in step `it` of (this tile) * (another held tile of the same shape)
    __device__ inline float dot_row(const TileRegs &o, int it) const {
        alignas(16) T a[VEC], b[VEC];
        *reinterpret_cast<uint4 *>(a) = v[it];
        *reinterpret_cast<uint4 *>(b) = o.v[it];
        float s = 0.f;
#pragma unroll
        for (int u = 0; u < VEC; ++u) s += to_f32(a[u]) * to_f32(b[u]);
        return s;
    }
    // sum over the TPR lanes that share a row (they are adjacent; the additions are those of a butterfly)
    __device__ static inline float row_sum(float x) {
        static_assert(TPR == 8 || TPR == 16 || TPR == 32, "lanes per row");
        x = lane_sum<(TPR < 16 ? TPR : 16)>(x);
        return TPR == 32 ? x + __shfl_xor(x, 16) : x;
    }
    // The query/key feature map of section 3.3 on the held tile, in place: every row x becomes
    // SiLU(x) / ||SiLU(x)||_2 (a row whose image is exactly zero, such as a row past the end, stays zero).
    // The TPR lanes that share a row are adjacent, so the row sum is a butterfly over them.
    // inv[it] = 1 / norm of the row held in step it (0 for a zero row).
    __device__ inline void feature_map(float (&inv)[NIT]) {
#pragma unroll
        for (int it = 0; it < NIT; ++it) {
            alignas(16) T e[VEC];
            *reinterpret_cast<uint4 *>(e) = v[it];
            float sv[VEC], ss = 0.f;
#pragma unroll
            for (int u = 0; u < VEC; ++u) { // every step an explicit single-rounding operation: all kernels get the same bits
                const float x = to_f32(e[u]);
                sv[u] = __fmul_rn(x, sigmoid_f32(x));
                ss = __fmaf_rn(sv[u], sv[u], ss);
            }
            ss = row_sum(ss);
            inv[it] = ss > 0.f ? __frsqrt_rn(ss) : 0.f;
#pragma unroll
            for (int u = 0; u < VEC; ++u) e[u] = from_f32<T>(__fmul_rn(sv[u], inv[it]));
            v[it] = *reinterpret_cast<const uint4 *>(e);
            __builtin_amdgcn_sched_barrier(0); // one step at a time: interleaved, the steps' temporaries do not fit
        }
    }
    // Gradient through the map, for a tile whose pre-activations x this object holds: src = dy in LDS
    // (same shape, leading dimension ld);
    //     dx = SiLU'(x) (dy - y (y . dy)) / ||SiLU(x)||,  SiLU'(x) = sig (1 + x (1 - sig)),  y = SiLU(x) / ||SiLU(x)||,
    // written to global memory (rows >= nvalid dropped).  A first pass forms the rows' norms and keeps every sigmoid (the
    // fast one: y need not have the bits of the mapped tile here); a row's sums are butterflies over its TPR lanes.
    __device__ inline void feature_map_bwd_store(const T *src, int ld, T *dst, long row_stride, int nvalid, int t = threadIdx.x) const {
        const int tr = t / TPR, tc = (t % TPR) * VEC;
        float sg[NIT][VEC], inv[NIT];
#pragma unroll
        for (int it = 0; it < NIT; ++it) {
            alignas(16) T x[VEC];
            *reinterpret_cast<uint4 *>(x) = v[it];
            float ss = 0.f;
#pragma unroll
            for (int u = 0; u < VEC; ++u) {
                const float xv = to_f32(x[u]);
                sg[it][u] = sigmoid_fast_f32(xv);
                const float sv = __fmul_rn(xv, sg[it][u]);
                ss = __fmaf_rn(sv, sv, ss);
            }
            ss = row_sum(ss);
            inv[it] = ss > 0.f ? __frsqrt_rn(ss) : 0.f;
        }
#pragma unroll
        for (int it = 0; it < NIT; ++it) {
            alignas(16) T x[VEC], a[VEC];
            *reinterpret_cast<uint4 *>(x) = v[it];
            *reinterpret_cast<uint4 *>(a) = *reinterpret_cast<const uint4 *>(src + (it * RPI + tr) * ld + tc);
            float y[VEC], dsl[VEC], dot = 0.f;
#pragma unroll
            for (int u = 0; u < VEC; ++u) {
                const float xv = to_f32(x[u]), s1 = sg[it][u];
                y[u] = __fmul_rn(__fmul_rn(xv, s1), inv[it]);
                dsl[u] = s1 * (1.f + xv * (1.f - s1)) * inv[it];
                dot += to_f32(a[u]) * y[u];
            }
            dot = row_sum(dot);
#pragma unroll
            for (int u = 0; u < VEC; ++u) a[u] = from_f32<T>((to_f32(a[u]) - y[u] * dot) * dsl[u]);
            if (it * RPI + tr < nvalid)
                *reinterpret_cast<uint4 *>(dst + (long)(it * RPI + tr) * row_stride + tc) = *reinterpret_cast<const uint4 *>(a);
            __builtin_amdgcn_sched_barrier(0);
        }
    }
    // held tile -> global memory (rows >= nvalid dropped)
    __device__ inline void store_global(T *dst, long row_stride, int nvalid, int t = threadIdx.x) const {
        const int tr = t / TPR, tc = (t % TPR) * VEC;
#pragma unroll
        for (int it = 0; it < NIT; ++it)
            if (it * RPI + tr < nvalid)
                *reinterpret_cast<uint4 *>(dst + (long)(it * RPI + tr) * row_stride + tc) = v[it];
    }
    // Per-row factors for scale_rows: f[it] = src[row held in step it] (rows of the tile this lane touches).
    __device__ inline void load_row_factors(float (&f)[NIT], const float *src, int t = threadIdx.x) const {
        const int tr = t / TPR;
#pragma unroll
        for (int it = 0; it < NIT; ++it) f[it] = src[it * RPI + tr];
    }
    // held tile <- diag(f) * tile, in the storage type
    __device__ inline void scale_rows(const float (&f)[NIT]) {
#pragma unroll
        for (int it = 0; it < NIT; ++it) {
            alignas(16) T e[VEC];
            *reinterpret_cast<uint4 *>(e) = v[it];
#pragma unroll
            for (int u = 0; u < VEC; ++u) e[u] = from_f32<T>(to_f32(e[u]) * f[it]);
            v[it] = *reinterpret_cast<const uint4 *>(e);
        }
    }
};
// ---------------------------------------------------------------------------------------------
// X = (I + A)^{-1} for a 64x64 strictly-lower-triangular A (section 3.2: the inverse of the unit
// lower-triangular matrix of Eq. 10 by forward substitution), blockwise, fp32 throughout.
// On entry sX (fp32, leading dimension ld, a multiple of 4) holds A in its three lower 32 x 32 blocks, the strictly lower
// part of the diagonal ones with zeros above; the upper right block need not hold anything.  On exit the diagonal blocks hold
// those of X, and the UPPER RIGHT block holds X21, the lower left block of X (whose own place is still being read as A21 by
// the other wave when a wave writes its columns; X itself is zero up there).
// The four 16x16 diagonal blocks are solved column by column by one wavefront (a lane per column), then 2x2 block merges
// X21 = -X22 (A21 X11) double the block size 16 -> 32 -> 64 on the fp32 matrix cores (16x16x4).  The contraction index of a
// merge is walked so that lane group g = lane >> 4 feeds k = 4 g + i in step i: an A operand is then 16 bytes of one row, and
// the accumulator of the inner product is, register by register, the B operand of the outer one, so it never leaves the
// registers.  That keeps the inverse at about 150 LDS instructions and one barrier (before its last stage, which
// two wavefronts share); merging on the vector ALU from LDS took about 800 and seven, and bound the whole prep kernel.
// Ends with a barrier.
__device__ inline f32x4 mfma16(f32x4 acc, float a, float b) { return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, acc, 0, 0, 0); }
// acc += A B for 16x16 blocks in LDS
__device__ inline void mma16_lds(f32x4 &acc, const float *A, const float *B, int ld) {
    const int lane = threadIdx.x & 63, j = lane & 15, g4 = 4 * (lane >> 4);
    const f32x4 a = *reinterpret_cast<const f32x4 *>(A + j * ld + g4);
#pragma unroll
    for (int i = 0; i < 4; ++i) acc = mfma16(acc, a[i], B[(g4 + i) * ld + j]);
}
// acc += A M for a 16x16 block in LDS and one in accumulator layout
__device__ inline void mma16_acc(f32x4 &acc, const float *A, const f32x4 &M, int ld) {
    const int lane = threadIdx.x & 63, j = lane & 15, g4 = 4 * (lane >> 4);
    const f32x4 a = *reinterpret_cast<const f32x4 *>(A + j * ld + g4);
#pragma unroll
    for (int i = 0; i < 4; ++i) acc = mfma16(acc, a[i], M[i]);
}
__device__ inline void acc16_store_neg(float *dst, const f32x4 &acc, int ld) {
    const int lane = threadIdx.x & 63, j = lane & 15, g4 = 4 * (lane >> 4);
#pragma unroll
    for (int i = 0; i < 4; ++i) dst[(g4 + i) * ld + j] = -acc[i];
}
__device__ inline void tri_inverse_64(float *sX, int ld) {
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    if (wave == 0) {
        float *blk = sX + (lane >> 4) * 16 * (ld + 1);
        const int j = lane & 15;
        float x[16];
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            float s = (i == j) ? 1.f : 0.f;
#pragma unroll
            for (int m0 = 0; m0 < i; m0 += 4) {
                const f32x4 a = *reinterpret_cast<const f32x4 *>(blk + i * ld + m0);
#pragma unroll
                for (int m = m0; m < m0 + 4 && m < i; ++m) s -= a[m - m0] * x[m];
            }
            x[i] = s;
        }
#pragma unroll
        for (int i = 0; i < 16; ++i) blk[i * ld + j] = x[i];
        // 16 -> 32, from what other lanes of this wavefront have just stored.  The hardware keeps a wavefront's LDS accesses in
        // order, so no barrier is needed; the compiler has to be told (per lane the addresses look unrelated).
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
        f32x4 m0 = {0.f, 0.f, 0.f, 0.f}, m1 = m0, y0 = m0, y1 = m0;
        float *d0 = sX, *d1 = sX + 32 * (ld + 1);
        mma16_lds(m0, d0 + 16 * ld, d0, ld);
        mma16_lds(m1, d1 + 16 * ld, d1, ld);
        mma16_acc(y0, d0 + 16 * (ld + 1), m0, ld);
        mma16_acc(y1, d1 + 16 * (ld + 1), m1, ld);
        acc16_store_neg(d0 + 16 * ld, y0, ld);
        acc16_store_neg(d1 + 16 * ld, y1, ld);
    }
    lds_barrier();
    if (wave < 2) { // 32 -> 64: wave n forms columns 16 n .. 16 n + 15
        const int n = wave;
        const float *A21 = sX + 32 * ld, *X22 = sX + 32 * (ld + 1);
        f32x4 m0 = {0.f, 0.f, 0.f, 0.f}, m1 = m0, y0 = m0, y1 = m0;
        if (n == 0) { // X11 is lower triangular
            mma16_lds(m0, A21, sX, ld);
            mma16_lds(m1, A21 + 16 * ld, sX, ld);
        }
        mma16_lds(m0, A21 + 16, sX + 16 * ld + 16 * n, ld);
        mma16_lds(m1, A21 + 16 * ld + 16, sX + 16 * ld + 16 * n, ld);
        mma16_acc(y0, X22, m0, ld); // so is X22
        mma16_acc(y1, X22 + 16 * ld, m0, ld);
        mma16_acc(y1, X22 + 16 * (ld + 1), m1, ld);
        acc16_store_neg(sX + 32 + 16 * n, y0, ld);
        acc16_store_neg(sX + 16 * ld + 32 + 16 * n, y1, ld);
    }
    lds_barrier();
}

} // namespace dn
