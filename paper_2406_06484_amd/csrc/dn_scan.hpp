// The chain-serial kernels: the forward scan over the chunks of a sequence, which carries the state S, and the reverse scan,
// which carries its gradient dS.
//
//   forward  X = V - K S;  Ut = T X (Eq. 8, 11: T V - (T K) S);  O = Q S + tril(Q K^T) Ut (Eq. 9);  S += K^T Ut (Eq. 8)
//   reverse  dUt = P^T dO + K dS';  dV = T^T dUt;  dS = dS' + Q^T dO - K^T dV
//
// The columns of the state are independent, so a wavefront owns 16 of them for a whole chain and the chain never leaves its
// registers.  With the 16 x 16 matrix instructions an accumulator holds, for lane l, column l & 15 and four rows of the lane
// group l >> 4; an operand holds index l & 15 and, per lane group, 16 bytes of consecutive contraction indices.  Rows of a
// product are handed to the accumulators in the order (row16 below) that makes those of a contraction step, rounded, exactly
// the operand of the product that follows: S -> K S -> T X -> K^T Ut -> S is four products without a store, a barrier or a
// lane exchange between them.  (The form this replaced kept 32 x 32 tiles of the state on eight wavefronts, formed W = T K and
// U = T V per chunk and passed S, W, P and Ut through the LDS: 5.8 K cycles a step in three barrier intervals, whose operand
// reads alone filled the LDS for 3 K of them.  Now 2.9 K beside one chain wave and 4.1 K beside four.)
// Scan times before and now, by events on one device: forward pass of 1 x 1000 tokens, 16 heads of 128, 34.7 -> 22.9 us; 8 x 2048 tokens of width 2048,
// d = 128, forward 85.9 -> 66.9, forward that keeps its tiles 102.3 -> 97.0, reverse 99.0 -> 85.1 (both at 5.2 TB/s: HBM bounds them); gated 147 -> 102
// and 112 -> 97; d = 256 229 -> 165 and 236 -> 136; 4 x 4096, d = 64, 123 -> 121 and 126 -> 112; fp32, 2 x 1500 tokens, 8 heads of 64, 184 -> 96 and 170 -> 97.
//
// A workgroup is NCW such chain waves (16 NCW columns) and four or eight helper waves (kSplitHelpers).  What bounds a chain wave is the rate at which ONE wave
// can read the LDS (24 cycles for 16 bytes a lane, 13 for 8; four waves together reach four times that), not its products (16
// cycles for each of those reads), so everything that is not on the chain goes to the helpers: they bring the tiles from global
// memory one or two chunks ahead (kScanSets), through registers into the LDS, form P = tril(Q K^T), keep it in registers as the operand of the
// next product, and form O (P^T dO) from it; in the forward scan a helper owns 16 tokens, whose Q no other wave reads.
// A chunk step is two barrier intervals; what an interval reads is written in the other one, so only K and the tables are kept twice.
//   forward  A  chain: X = V - K S, Ut = T X                helpers: P, Q S
//            B  chain: S += K^T Ut                          helpers: O = Q S + P Ut, O to memory, the next chunk's K, V, T, Q
//   reverse  A  chain: K dS', Q^T dO                        helpers: P, P^T dO, (fp32) Q^T dO, this chunk's T, the dV of the chunk before to memory
//            B  chain: dUt, dV = T^T dUt, dS -= K^T dV      helpers: the next chunk's K, Q, dO
//
// Rounding points in bf16: S, Ut, P, T (dS', dV) as operands; X and dUt go in as two of them (kTwoTerms).  The diagonal of T, the largest
// term of a row of T X, is not in the tile: Ut = beta X + (T - diag(beta)) X with the fp32 beta and X; in the same way dV = T^T dUt.
#pragma once
#include <type_traits>
#include <utility>

#include "dn_device.hpp"
#include "dn_host.hpp"

namespace dn {

constexpr int NTL = 256; // helper threads of a scan workgroup

// ---- 16 x 16 products --------------------------------------------------------------------------------------------------
// VEC: contraction indices per lane and operand; KS = 4 VEC: contraction length of one operand; TPS: accumulator tiles whose
// rows make up one operand
template <typename T> struct Op;
template <> struct Op<bf16> { typedef bf16x8 frag; static constexpr int VEC = 8, KS = 32, TPS = 2; };
template <> struct Op<float> { typedef f32x4 frag; static constexpr int VEC = 4, KS = 16, TPS = 1; };

__device__ inline void mma16(f32x4 &acc, const bf16x8 &a, const bf16x8 &b) { acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, acc, 0, 0, 0); }
__device__ inline void mma16(f32x4 &acc, const f32x4 &a, const f32x4 &b) {
#pragma unroll
    for (int i = 0; i < 4; ++i) acc = mfma16(acc, a[i], b[i]);
}
// the matrix row that stands in row m of accumulator tile t; row4: the first of the four rows of lane group g
template <typename T> __host__ __device__ constexpr int row16(int t, int m) {
    return Op<T>::TPS == 2 ? 32 * (t >> 1) + 8 * (m >> 2) + (m & 3) + 4 * (t & 1) : 16 * t + m;
}
template <typename T> __host__ __device__ constexpr int row4(int t, int g) { return row16<T>(t, 4 * g); }
// contraction step s of the operand that the accumulator tiles of a product make
__device__ inline bf16x8 as_operand(const f32x4 *t, int s, bf16) {
    bf16x8 f;
#pragma unroll
    for (int i = 0; i < 4; ++i) { f[i] = (bf16)t[2 * s][i]; f[4 + i] = (bf16)t[2 * s + 1][i]; }
    return f;
}
__device__ inline f32x4 as_operand(const f32x4 *t, int s, float) { return t[s]; }
// ... of what the rounding left out of it (bf16; fp32 operands are not rounded)
__device__ inline bf16x8 rest_operand(const f32x4 *t, const bf16x8 &rounded, int s) {
    bf16x8 f;
#pragma unroll
    for (int i = 0; i < 4; ++i) { f[i] = (bf16)(t[2 * s][i] - (float)rounded[i]); f[4 + i] = (bf16)(t[2 * s + 1][i] - (float)rounded[4 + i]); }
    return f;
}
__device__ inline f32x4 rest_operand(const f32x4 *, const f32x4 &, int) { return f32x4{0.f, 0.f, 0.f, 0.f}; }
__device__ inline f32x4 zero4() { return f32x4{0.f, 0.f, 0.f, 0.f}; }

// ---- LDS tiles ---------------------------------------------------------------------------------------------------------
// Rows without padding; the 16-byte pieces of a row are permuted by an XOR with a function of the row, chosen so that the
// rows of one operand (row16 order, one piece per lane), the transposing reads (four rows, four pieces) and plain rows each
// spread over all 64 banks: 4 cycles for each of the two kinds of read (in rows padded by 16 or 32 bytes one of the two, or both, take 8).
template <typename T, int COLS> struct LdsTile {
    static constexpr int RB = COLS * (int)sizeof(T), SLOTS = RB / 16, VEC = Op<T>::VEC;
    static constexpr int bytes = C * RB;
    __device__ static int swz(int r) {
        if (sizeof(T) == 2) {
            const int h = (0 - (r >> 3)) & 3;
            return SLOTS >= 16 ? ((r & 3) << 2) | h : SLOTS == 8 ? ((r & 2) << 1) | h : 0;
        }
        return SLOTS >= 16 ? r & 15 : SLOTS == 8 ? (r >> 1) & 7 : SLOTS == 4 ? (r >> 2) & 3 : 0;
    }
    __device__ static int at(int r, int piece) { return r * RB + ((piece ^ swz(r)) << 4); }
    // operands with the contraction index along the rows: row row16(t, l & 15), piece 4 s + (l >> 4)
    __device__ static int kc0(int lane) { const int r = row16<T>(0, lane & 15); return at(r, lane >> 4); }
    __device__ static int kc(int kc0, int t, int s) { return (kc0 ^ (s << 6)) + row16<T>(t, 0) * RB; }
    // ... across the rows: index row16(t, l & 15) along the row, contraction rows KS s + VEC (l >> 4) + 0 .. VEC - 1
    __device__ static int ks0(int lane) {
        const int i = lane & 15, g = lane >> 4;
        if (sizeof(T) == 2) { const int r = 8 * g + (i >> 2); return at(r, i & 3); }
        return at(4 * g, i >> 2) + 4 * (i & 3);
    }
    // accumulator-shaped reads: column 16 c + (l & 15), rows row4(t, l >> 4) + 0 .. 3
    __device__ static int ac0(int lane, int c) {
        const int i = lane & 15, g = lane >> 4;
        if (sizeof(T) == 2) { const int r = 8 * g + (i >> 2); return at(r, 2 * c + ((i & 3) >> 1)) + 8 * (i & 1); }
        return 0; // (see read_ac)
    }
};
__device__ inline s16x4 lds_tr(const unsigned char *p) {
    typedef __attribute__((address_space(3))) s16x4 lds_s16x4;
    return __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4 *)(p));
}
template <typename T, int COLS> __device__ inline typename Op<T>::frag read_kc(const unsigned char *tile, int kc0, int t, int s) {
    return *reinterpret_cast<const typename Op<T>::frag *>(tile + LdsTile<T, COLS>::kc(kc0, t, s));
}
template <typename T, int COLS> __device__ inline typename Op<T>::frag read_ks(const unsigned char *tile, int ks0, int t, int s) {
    using L = LdsTile<T, COLS>;
    if constexpr (sizeof(T) == 2) {
        const unsigned char *p = tile + (ks0 ^ ((t >> 1) << 6)) + 32 * s * L::RB + 8 * (t & 1);
        const s16x4 lo = lds_tr(p), hi = lds_tr(p + 4 * L::RB);
        return __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
    } else {
        f32x4 f;
#pragma unroll
        for (int i = 0; i < 4; ++i) f[i] = *reinterpret_cast<const float *>(tile + (ks0 ^ (t << 6) ^ (L::swz(i) << 4)) + (16 * s + i) * L::RB);
        return f;
    }
}
// fp32: products that meet a larger term are summed from zero and added at the end, which keeps every partial sum's rounding
// to its own size (summed onto V, S and dS the results are 10 to 60 % further from the exact ones); bf16 rounds their sum to 8 bits anyway.
// The sums over T^T walk the tokens from the chunk's end: the near ones, whose terms are the large ones, then the diagonal (from its near end,
// where keys and queries are alike, the large terms stand in the partial sum while the rest is added, and dv is 31 % further off)
template <typename T> constexpr bool kSumFirst = sizeof(T) == 4;
// bf16: X and dUt, the right factors of the products with T and T^T, as two bf16 operands, the rounded value and the rest, that
// meet the same reads of T (six more products each).  Where keys are alike X = V - K S and dV are differences of large terms, and a
// factor rounded to 8 bits in between was 9 to 20 % of error in o, 15 to 20 in the state, 7 to 8 in dv and 13 to 23 in dbeta (mean cosine of
// the keys 0.8 to 0.9, against products that take V and dUt apart); with the second term every tensor is below those products.  It costs 1.3 us
// of 26.7 (1 x 1000 tokens, 16 heads of 128), 2 of 68 (forward scan, 8 x 2048) and 2 of 82 (reverse scan).
template <typename T> constexpr bool kTwoTerms = sizeof(T) == 2;
// four elements of accumulator tile t in storage format
template <typename T, int COLS> __device__ inline auto read_ac(const unsigned char *tile, int ac0, int t, int lane, int c) {
    using L = LdsTile<T, COLS>;
    if constexpr (sizeof(T) == 2) return lds_tr(tile + ac0 + row16<T>(t, 0) * L::RB);
    else {
        f32x4 f;
#pragma unroll
        for (int i = 0; i < 4; ++i) f[i] = *reinterpret_cast<const float *>(tile + L::at(row4<T>(t, lane >> 4) + i, 4 * c + ((lane & 15) >> 2)) + 4 * (lane & 3));
        return f;
    }
}
__device__ inline f32x4 widen(const s16x4 &x) {
    f32x4 f;
#pragma unroll
    for (int i = 0; i < 4; ++i) f[i] = __uint_as_float((unsigned)(unsigned short)x[i] << 16);
    return f;
}
__device__ inline f32x4 widen(const f32x4 &x) { return x; }
__device__ inline bf16x8 join(const s16x4 *x, int s) { return __builtin_bit_cast(bf16x8, __builtin_shufflevector(x[2 * s], x[2 * s + 1], 0, 1, 2, 3, 4, 5, 6, 7)); }
__device__ inline f32x4 join(const f32x4 *x, int s) { return x[s]; }

// N operand reads ld(0) .. ld(N - 1), DEPTH of them in flight ahead of the products mm(i, operand) that use them; the numbers are
// compile-time constants (std::integral_constant)
template <int I> using Num = std::integral_constant<int, I>;
template <int N, int D, int I, typename F, typename LD, typename MM> __device__ __forceinline__ void stream_one(F (&a)[D], LD &ld, MM &mm) {
    mm(Num<I>{}, a[I % D]);
    if constexpr (I + D < N) a[I % D] = ld(Num<I + D>{});
}
template <int N, int D, typename F, typename LD, typename MM, int... I> __device__ __forceinline__ void stream_all(F (&a)[D], LD &ld, MM &mm, std::integer_sequence<int, I...>) {
    (stream_one<N, D, I>(a, ld, mm), ...);
}
template <int D, typename F, typename LD, int... I> __device__ __forceinline__ void stream_ahead(F (&a)[D], LD &ld, std::integer_sequence<int, I...>) {
    ((a[I] = ld(Num<I>{})), ...);
}
template <int N, int DEPTH, typename F, typename LD, typename MM> __device__ __forceinline__ void stream(LD ld, MM mm) {
    constexpr int D = DEPTH < N ? DEPTH : N;
    F a[D];
    stream_ahead<D>(a, ld, std::make_integer_sequence<int, D>{});
    __builtin_amdgcn_sched_barrier(0); // (the compiler would move the reads down to their uses)
    stream_all<N, D>(a, ld, mm, std::make_integer_sequence<int, N>{});
}
// The non-zero (tile, contraction step) pairs of a C x C triangle, steps outermost: pair e of the lower one (row blocks of one
// contraction step: TPS tiles) and of the upper one
struct TilePair { int t, s; };
template <int NC, int TPS> __host__ __device__ constexpr TilePair lower_pair(int e) {
    int s = 0;
    while (e >= (NC - s) * TPS) { e -= (NC - s) * TPS; ++s; }
    return {s * TPS + e, s};
}
template <int TPS> __host__ __device__ constexpr TilePair upper_pair(int e) {
    int s = 0;
    while (e >= (s + 1) * TPS) { e -= (s + 1) * TPS; ++s; }
    return {e, s};
}
// acc[pair(e).t] += f[e] b[pair(e).s] for every e
template <typename F, typename PAIR, int... I> __device__ __forceinline__ void second_terms(f32x4 *acc, const F *f, const F *b, PAIR pair, std::integer_sequence<int, I...>) {
    (mma16(acc[pair(Num<I>{}).t], f[I], b[pair(Num<I>{}).s]), ...);
}

// ---- pieces of a tile between global memory, registers and the LDS ------------------------------------------------------
// A 64 x COLS tile as 16-byte pieces, piece numbers t, t + NTL, ... of thread t; consecutive threads hold consecutive pieces.
// Requests of rows at or past nvalid return zeros and touch no memory: the descriptor's range ends at that row, or (SELECT) their lanes
// point past a range that does not depend on the chunk.  No branch stands around a request, and the compiler knows how many are in
// flight.  Which form: forward scan that keeps its tiles, 8 x 2048 tokens of 16 heads of 128, 106 us with the select and 101 without,
// reverse scan 87 and 91 (d = 256: 157 and 168).
template <typename T, int COLS> struct Pieces {
    using L = LdsTile<T, COLS>;
    static constexpr int PPR = L::SLOTS, N = C * PPR, NIT = (N + NTL - 1) / NTL;
    static_assert(N % NTL == 0 || N < NTL, "whole rounds");
    uint4 v[NIT];
    template <int AUX, bool SELECT = false> __device__ __forceinline__ void load(const T *src, long row_stride, int nvalid, int t) {
        const int stride = (int)row_stride * (int)sizeof(T);
        const __amdgpu_buffer_rsrc_t rs = make_rsrc(src, SELECT ? kBufRange : nvalid * stride);
#pragma unroll
        for (int it = 0; it < NIT; ++it) {
            const int e = it * NTL + t, r = e / PPR, p = e % PPR;
            v[it] = buf_load16<AUX>(rs, !SELECT || r < nvalid ? r * stride + 16 * p : kBufRange, 0);
        }
    }
    // SIGN: with the sign of every element flipped
    template <bool SIGN = false> __device__ __forceinline__ void store(unsigned char *tile, int t) const {
        constexpr unsigned S = !SIGN ? 0u : sizeof(T) == 2 ? 0x80008000u : 0x80000000u;
#pragma unroll
        for (int it = 0; it < NIT; ++it) {
            const int e = it * NTL + t, r = e / PPR, p = e % PPR;
            if (N >= NTL || t < N) *reinterpret_cast<uint4 *>(tile + L::at(r, p)) = make_uint4(v[it].x ^ S, v[it].y ^ S, v[it].z ^ S, v[it].w ^ S);
        }
    }
    // rows times f, in the storage type
    __device__ __forceinline__ void scale(const float (&f)[NIT]) {
        constexpr int VEC = Op<T>::VEC;
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
// LDS tile -> global rows (rows at or past nvalid are dropped: their lanes point past the descriptor's range)
template <typename T, int COLS, int AUX> __device__ __forceinline__ void tile_out(T *dst, long row_stride, int nvalid, const unsigned char *tile, int t) {
    using P = Pieces<T, COLS>;
    const int stride = (int)row_stride * (int)sizeof(T);
    const __amdgpu_buffer_rsrc_t rs = make_rsrc(dst);
#pragma unroll
    for (int it = 0; it < P::NIT; ++it) {
        const int e = it * NTL + t, r = e / P::PPR, p = e % P::PPR;
        const u32x4 x = *reinterpret_cast<const u32x4 *>(tile + P::L::at(r & (C - 1), p));
        __builtin_amdgcn_raw_buffer_store_b128(x, rs, r < nvalid ? r * stride + 16 * p : kBufRange, 0, AUX);
    }
}

// The S, dS' and Ut tiles in the workspace stand in the order of the operands: for every 16 columns of d_v and every
// contraction step s (over d_k, or over the chunk's tokens for Ut) the 16 bytes of lane l at 16 frag_place(l).  They leave from registers in
// whole kilobytes.  In bf16 up to d_k = 128 the chunk kernel reads its operands from the tile as it stands here (dn_chunk_bf16.hpp); the
// lanes are permuted so that these reads find different banks of the LDS.
template <typename T, int ROWS> __device__ inline T *frag_tile(void *ws, long tile, int dv, int col16) {
    return (T *)ws + (tile * dv + 16 * col16) * ROWS;
}
template <typename T, int DK> __device__ inline int frag_place(int lane) { return sizeof(T) == 2 && DK <= 128 ? lane ^ (lane >> 4 << 2) : lane; }
template <typename T> __device__ inline void store_frag(T *tile, int s, const typename Op<T>::frag &f, int place) {
    __builtin_nontemporal_store(__builtin_bit_cast(u32x4, f), reinterpret_cast<u32x4 *>(tile) + 64 * s + place);
}

// ---- shared by the two scans -------------------------------------------------------------------------------------------
// Workgroup ids are laid out so that the column blocks of one chain land on the same XCD (ids are dealt round-robin over the 8
// XCDs) and share its L2 for the Q, K, T tiles they all read.
__device__ inline bool chain_of_block(int bid, int nchains, int nv, int &chain, int &vbi) {
    const int xcd = bid & 7, slot = bid >> 3;
    vbi = slot % nv;
    chain = (slot / nv) * 8 + xcd;
    return chain < nchains;
}
__host__ inline int chain_grid(int nchains, int nv) { return ((nchains + 7) / 8) * 8 * nv; }

// Up to d_k = 128 the helpers are eight waves, four that form P and the products with it and four that move tiles; with the
// registers of d_k = 256 a SIMD holds only two waves, and four do both.  (The forward scans without outputs form nothing: there the first four wait at
// the barriers.  They share a grid, and so the number of threads, with the reverse scan.)
// So they do in the fp32 forward scan that has outputs: with eight it takes 79 us and not 99 (3 x 1500 tokens, 8 heads of 64), but the
// reverse scan, whose chain waits for the helpers' products, takes 97 with eight, and it is held to the forward scan's time
// (tests/test_gpu_scan_balance.py).
enum { DIR_FWD = 0, DIR_BWD = 1 };
template <typename T, int DK, int DIR> constexpr bool kSplitHelpers = DK <= 128 && (sizeof(T) == 2 || DIR == DIR_BWD);
// fp32, whose products and not its LDS reads are what a wave waits for: Q^T dO by the helpers that move tiles (in bf16 it gains nothing)
template <typename T> constexpr bool kOffloadQdO = sizeof(T) == 4;
template <typename T, int DK, int NCW> struct ScanSmem {
    static constexpr int BV = 16 * NCW;
    static constexpr size_t szK = LdsTile<T, DK>::bytes, szV = LdsTile<T, BV>::bytes, szC = LdsTile<T, C>::bytes;
    static constexpr size_t szTab = 3 * C * sizeof(float); // per chunk parity: gamma_i, 1 / gamma_i, -beta_i
    static constexpr size_t oK = 0, oQ = 2 * szK, oV = oQ + (szK > szV ? szK : szV), oT = oV + szV, oTab = oT + szC, oX = oTab + 2 * szTab;
    // forward: S and Ut as operands, chain waves to helpers (Q: every helper's own rows, then the rows of O)
    static constexpr size_t szS = (size_t)DK * BV * sizeof(T), oS = oX, oU = oS + szS, fwd_bytes = oU + szV;
    // reverse: P^T dO (and Q^T dO) as accumulators, helpers to chain waves; dV
    static constexpr size_t oE = oX, oF = oE + (size_t)C * BV * sizeof(float), oO = oF + (kOffloadQdO<T> ? (size_t)DK * BV * sizeof(float) : 0), bwd_bytes = oO + szV;
    static constexpr size_t bytes = fwd_bytes > bwd_bytes ? fwd_bytes : bwd_bytes;
};
// Number of a helper wave: 0 .. 3 form, 4 .. 7 move (where four do both: 0 .. 3).  Waves are dealt to the four SIMDs in turn; the ones that
// share theirs with a chain wave move tiles, as far as there are others to do the forming.
template <typename T, int DK, int DIR, int NCW> __device__ inline int helper_number(int wave) {
    if (!kSplitHelpers<T, DK, DIR>) return wave & 3;
    if (NCW == 1) return wave == 4 ? 6 : wave == 8 ? 7 : wave < 4 ? wave - 1 : wave - 2;
    if (NCW == 2) return ((wave & 2) ? (wave & 1) + (wave >> 1 & 2) : 4 + (wave & 1) + (wave >> 2 & 2));
    return wave - NCW;
}
template <typename T, int DK, int DIR, int NCW> constexpr int kScanThreads = 64 * NCW + (kSplitHelpers<T, DK, DIR> ? 2 : 1) * NTL;
// How many chunks the helpers' registers hold on their way to the LDS: two (16 384 tokens of 8 heads of 256: forward scan that keeps its
// tiles 196 us with one and 168 with two, reverse scan 155 and 137); in fp32, whose steps are long and whose tiles are twice as large, one.
template <typename T> constexpr int kScanSets = sizeof(T) == 4 ? 1 : 2;
// what one chunk's row of the tables is made from, per thread lt < 64 (the others hold copies)
template <typename T, bool GATED> struct TabRegs {
    float gm, gi;
    T beta;
    __device__ __forceinline__ void load(const Ptrs &p, long row0, long tile, int H, int h, int nvalid, int lt) {
        const int i = lt & (C - 1);
        beta = ((const T *)p.beta)[(row0 + min(i, max(nvalid - 1, 0))) * H + h];
        if (GATED) { gm = p.gam[tile * 2 * C + i]; gi = p.gam[tile * 2 * C + C + i]; }
    }
    __device__ __forceinline__ void store(float *tab, bool pro, int nvalid, int lt) const {
        if (lt < C) {
            if (GATED) { tab[lt] = gm; tab[C + lt] = gi; }
            tab[2 * C + lt] = lt < nvalid ? 0.f - (pro ? sigmoid_f32(to_f32(beta)) : to_f32(beta)) : 0.f;
        }
    }
};
__device__ inline f32x4 tab4(const float *tab, int r) { return *reinterpret_cast<const f32x4 *>(tab + r); }
// The rows of P = tril(Q K^T) (TRANSPOSED: of P^T) in tile w, as operands: `own` = these rows of Q (of K), the other matrix from the
// LDS; contraction step c of the product that follows is formed if bit c of `blocks` is set
template <typename T, int DK, bool TRANSPOSED> __device__ __forceinline__ void form_p(typename Op<T>::frag (&pb)[C / Op<T>::KS], const typename Op<T>::frag (&own)[DK / Op<T>::KS],
                                                                                       const unsigned char *others, int w, int blocks, int lane) {
    using O = Op<T>;
    typedef typename O::frag frag;
    constexpr int NK = DK / O::KS, NC = C / O::KS, TPS = O::TPS, DEPTH = sizeof(T) == 4 ? 4 : 8;
    const int m = lane & 15, g = lane >> 4;
    const int kc = LdsTile<T, DK>::kc0(lane);
    const int i = (TPS == 2 ? 32 * (w >> 1) + 4 * (w & 1) : 16 * w) + row16<T>(0, m); // (w is not a compile-time value)
#pragma unroll
    for (int c = 0; c < NC; ++c) {
        f32x4 acc[TPS];
#pragma unroll
        for (int u = 0; u < TPS; ++u) acc[u] = zero4();
        if ((blocks >> c) & 1) {
            stream<TPS * NK, DEPTH, frag>([&](auto E) __attribute__((always_inline)) { return read_kc<T, DK>(others, kc, c * TPS + E % TPS, E / TPS); },
                                          [&](auto E, const frag &f) __attribute__((always_inline)) { mma16(acc[E % TPS], f, own[E / TPS]); });
            if (c == w / TPS)
#pragma unroll
                for (int u = 0; u < TPS; ++u)
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        const int j = row4<T>(c * TPS + u, g) + e;
                        acc[u][e] = (TRANSPOSED ? j >= i : j <= i) ? acc[u][e] : 0.f;
                    }
        }
        pb[c] = as_operand(acc, 0, T());
    }
}
// Operands from one wave to another, as registers: operand (or accumulator tile) number n of a region, 16 bytes a lane
template <typename F> __device__ inline F take(const unsigned char *region, int n, int lane) { return *reinterpret_cast<const F *>(region + (n * 64 + lane) * 16); }
template <typename F> __device__ inline void hand(unsigned char *region, int n, int lane, const F &f) { *reinterpret_cast<F *>(region + (n * 64 + lane) * 16) = f; }
// lanes of a wavefront that exchange data through the LDS: the hardware keeps a wavefront's accesses in order, the compiler has to be told
__device__ inline void wave_exchange() {
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

// The 16 rows (tokens row16(w, 0 .. 15)) of a 64 x COLS matrix that helper wave w owns: global memory <-> registers <-> the
// wave's own 16 rows of LDS (permuted as in LdsTile, whose function depends on the place within the tile only)
template <typename T, int COLS> struct OwnRows {
    using L = LdsTile<T, COLS>;
    static constexpr int PPR = L::SLOTS, N = 16 * PPR, NIT = (N + 63) / 64;
    uint4 v[NIT];
    __device__ static int at(int n, int piece) { return n * L::RB + ((piece ^ L::swz(row16<T>(0, n))) << 4); }
    __device__ static int token(int w, int n) { return (Op<T>::TPS == 2 ? 32 * (w >> 1) + 4 * (w & 1) : 16 * w) + row16<T>(0, n); }
    template <int AUX> __device__ __forceinline__ void load(const T *src, long row_stride, int nvalid, int w, int lane) {
        const int stride = (int)row_stride * (int)sizeof(T);
        const __amdgpu_buffer_rsrc_t rs = make_rsrc(src, nvalid * stride);
#pragma unroll
        for (int it = 0; it < NIT; ++it) {
            const int e = it * 64 + lane, n = e / PPR & 15, p = e % PPR;
            v[it] = buf_load16<AUX>(rs, N % 64 == 0 || e < N ? token(w, n) * stride + 16 * p : kBufRange, 0);
        }
    }
    __device__ __forceinline__ void store(unsigned char *mine, int lane) const {
#pragma unroll
        for (int it = 0; it < NIT; ++it) {
            const int e = it * 64 + lane;
            if (N % 64 == 0 || e < N) *reinterpret_cast<uint4 *>(mine + at(e / PPR, e % PPR)) = v[it];
        }
    }
    template <int AUX> __device__ static __forceinline__ void out(T *dst, long row_stride, int nvalid, const unsigned char *mine, int w, int lane) {
        const int stride = (int)row_stride * (int)sizeof(T);
        const __amdgpu_buffer_rsrc_t rs = make_rsrc(dst, nvalid * stride);
#pragma unroll
        for (int it = 0; it < NIT; ++it) {
            const int e = it * 64 + lane, n = e / PPR & 15, p = e % PPR;
            const u32x4 x = *reinterpret_cast<const u32x4 *>(mine + at(n, p));
            __builtin_amdgcn_raw_buffer_store_b128(x, rs, N % 64 == 0 || e < N ? token(w, n) * stride + 16 * p : kBufRange, 0, AUX);
        }
    }
};

// ---- forward -----------------------------------------------------------------------------------------------------------
// MODE = SCAN_OUT writes O and the final state; SCAN_STORE (the backward's recompute pass) writes every chunk-initial state and
// Ut to the workspace instead of O; SCAN_BOTH (a forward pass whose backward pass will not recompute) does both; SCAN_STATE
// writes only the final state (the first pass of a forward pass that is split over segments of the sequence, see k_scan_state).
enum { SCAN_OUT = 0, SCAN_STORE = 1, SCAN_BOTH = 2, SCAN_STATE = 3 };

template <typename T, int DK, int DV, int MODE, bool GATED, int NCW>
__device__ __forceinline__ void scan_fwd_body(const SeqMap &sm, int H, const Ptrs &p, int bid) {
    using SM = ScanSmem<T, DK, NCW>;
    using O = Op<T>;
    typedef typename O::frag frag;
    constexpr int BV = SM::BV, NV = DV / BV, TPS = O::TPS;
    constexpr int NKT = DK / 16, NK = DK / O::KS, NCT = C / 16, NC = C / O::KS; // tiles, contraction steps over d_k and over the chunk
    constexpr bool OUT = MODE == SCAN_OUT || MODE == SCAN_BOTH;
    constexpr int DIR = OUT ? DIR_FWD : DIR_BWD; // (the others share a launch with the reverse scan)
    constexpr bool SAVE = MODE == SCAN_STORE || MODE == SCAN_BOTH;
    // a workgroup's rows of V and O are whole 128-byte lines: non-temporal; with narrower column blocks a line is shared with
    // the neighbouring workgroup of the chain and keeps the default policy
    constexpr int kAuxV = BV * sizeof(T) >= 128 ? kAuxOnce : kAuxKeep;
    extern __shared__ __align__(16) unsigned char smem[];
    unsigned char *sQ = smem + SM::oQ, *sV = smem + SM::oV, *sT = smem + SM::oT, *sS = smem + SM::oS, *sU = smem + SM::oU;

    int chain, vbi;
    if (!chain_of_block(bid, sm.N * H, NV, chain, vbi)) return;
    int n = chain / H;
    const int h = chain - n * H, vb = vbi * BV;
    if (sm.order) { n = sm.order[n]; chain = n * H + h; } // packed: longest sequences first
    int t0, len, cb;
    sm.seq(n, t0, len, cb);
    const int nchunks = (len + C - 1) / C;
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6), lane = threadIdx.x & 63;

    // ---- helpers.  FORMS: P and O of the 16 tokens of tile w in every chunk; MOVES: K, V, T into the LDS
    const int hw = helper_number<T, DK, DIR, NCW>(wave);
    auto helper = [&](auto forms, auto moves) __attribute__((always_inline)) {
        constexpr bool FORMS = OUT && decltype(forms)::value, MOVES = decltype(moves)::value;
        int lane = threadIdx.x & 63, lt = 64 * (hw & 3) + lane;
        // helpers 0 and 3 (beside one chain wave: on the same SIMD) or 0 and 2, 1 and 3 get a long row of blocks and a short one
        const int w = !FORMS ? hw & 3 : NCW == 1 ? (hw == 0 ? 0 : 4 - hw) & 3 : hw < 2 ? hw : 5 - hw;
        // (d_k = 256: the addresses derived from these are formed where they are used, not carried through the loop; no registers)
        auto fresh = [&]() __attribute__((always_inline)) { if (DK > 128) asm volatile("" : "+v"(lt), "+v"(lane)); };
        constexpr int SETS = kScanSets<T>;
        struct Set { Pieces<T, DK> k; Pieces<T, BV> v; Pieces<T, C> t; OwnRows<T, DK> q; } r[SETS];
        TabRegs<T, GATED> tb[2];
        unsigned char *mine = sQ + w * 16 * (BV > DK ? LdsTile<T, BV>::RB : LdsTile<T, DK>::RB);
        auto nv_of = [&](int ic) __attribute__((always_inline)) { return ic < nchunks ? min(C, len - ic * C) : 0; };
        auto fetch = [&](Set &x, int ic) __attribute__((always_inline)) {
            const int nvalid = nv_of(ic), ii = min(ic, nchunks - 1);
            const long row0 = (long)t0 + (long)ii * C, tile = (long)(cb + ii) * H + h;
            if (MOVES) {
                x.k.template load<kAuxKeep>((const T *)p.k + (row0 * H + h) * DK, (long)H * DK, nvalid, lt);
                // (the transition-matrix pass of k_scan_state runs on v = 0: no row is valid)
                x.v.template load<kAuxV>((const T *)p.v + (row0 * H + h) * DV + vb, (long)H * DV, (MODE == SCAN_STATE && p.unit_state) ? 0 : nvalid, lt);
                x.t.template load<kAuxKeep>((const T *)p.Tm + tile * C * C, C, ic < nchunks ? C : 0, lt);
            }
            if (FORMS) x.q.template load<kAuxKeep>((const T *)p.q + (row0 * H + h) * DK, (long)H * DK, nvalid, w, lane);
        };
        auto tab_of = [&](int ic) __attribute__((always_inline)) { return reinterpret_cast<float *>(smem + SM::oTab + (ic & 1) * SM::szTab); };
        auto fetch_tab = [&](TabRegs<T, GATED> &x, int ic) __attribute__((always_inline)) {
            const int ii = min(ic, nchunks - 1);
            if (MOVES) x.load(p, (long)t0 + (long)ii * C, (long)(cb + ii) * H + h, H, h, min(C, len - ii * C), lt);
        };
        auto store_tab = [&](const TabRegs<T, GATED> &x, int ic) __attribute__((always_inline)) { if (MOVES) x.store(tab_of(ic), p.pro, nv_of(ic), lt); };
        frag q[NK];
        // V and T go to the LDS with their signs flipped: the chain forms K S - V and multiplies it by -T
        auto stash = [&](const Set &x, int ic) __attribute__((always_inline)) {
            if (MOVES) {
                x.k.store(smem + SM::oK + (ic & 1) * SM::szK, lt);
                x.v.template store<true>(sV, lt);
                x.t.template store<true>(sT, lt);
            }
            if (FORMS) {
                x.q.store(mine, lane);
                wave_exchange();
#pragma unroll
                for (int s = 0; s < NK; ++s) q[s] = *reinterpret_cast<const frag *>(mine + OwnRows<T, DK>::at(lane & 15, 4 * s + (lane >> 4)));
            }
        };
        fetch_tab(tb[0], 0); fetch_tab(tb[1], 1);
        fetch(r[0], 0);
        store_tab(tb[0], 0);
        stash(r[0], 0);
        // The second chunk is not asked for before the first one is there: past one round of the chip all workgroups of a round begin
        // together, and the first step waits for both chunks of all of them.  64 x 128 tokens of width 2048, d = 64 and 128: forward that keeps its
        // tiles 59.0 -> 55.3 and 77.6 -> 71.8 us, reverse 60.6 -> 53.9 and 74 -> 69.5, pair 100 -> 94 and 136 -> 130; few or long chains do not change.
        __builtin_amdgcn_sched_barrier(0);
        fetch_tab(tb[0], 2);
        fetch(r[SETS - 1], 1);
        lds_barrier();
        if (GATED) lds_barrier(); // (the chain waves read the tables before they hand over the state)
        auto step = [&](Set &nx, Set &cu, TabRegs<T, GATED> &nt, int ic) __attribute__((always_inline)) { // nx, nt: of chunk ic + 1
            fresh();
            store_tab(nt, ic + 1); // (bf16 up to d = 128: as compiled, every second step waits here for all that is under way, not only for the table)
            fetch_tab(nt, ic + 3);
            if (SETS == 2) fetch(cu, ic + 2); // (here rather than in B, where the LDS takes the next chunk)
            f32x4 o[NCW]; // O^T: lane = token, rows = 16 columns of the state per chain wave
            frag pb[NC];
            if constexpr (FORMS) {
                form_p<T, DK, false>(pb, q, smem + SM::oK + (ic & 1) * SM::szK, w, (2 << w / TPS) - 1, lane);
#pragma unroll
                for (int c = 0; c < NCW; ++c) o[c] = zero4();
                stream<NCW * NK, 8, frag>([&](auto E) __attribute__((always_inline)) { return take<frag>(sS, (E % NCW) * NK + E / NCW, lane); },
                                          [&](auto E, const frag &f) __attribute__((always_inline)) { mma16(o[E % NCW], f, q[E / NCW]); });
            }
            lds_barrier();
            fresh();
            if constexpr (FORMS) {
                const int m = lane & 15, g = lane >> 4;
                stream<NCW * NC, 8, frag>([&](auto E) __attribute__((always_inline)) { return take<frag>(sU, (E % NCW) * NC + E / NCW, lane); },
                                          [&](auto E, const frag &f) __attribute__((always_inline)) { mma16(o[E % NCW], f, pb[E / NCW]); });
                float gm = 1.f;
                if (GATED) gm = tab_of(ic)[OwnRows<T, BV>::token(w, m)]; // o_i = gamma_i o~_i
#pragma unroll
                for (int c = 0; c < NCW; ++c) {
                    if (GATED) o[c] *= gm;
                    const int byte = (16 * c + 4 * g) * (int)sizeof(T);
                    st4(reinterpret_cast<T *>(mine + OwnRows<T, BV>::at(m, byte >> 4) + (byte & (16 - 4 * (int)sizeof(T)))), o[c][0], o[c][1], o[c][2], o[c][3]);
                }
                wave_exchange();
                OwnRows<T, BV>::template out<kAuxV>((T *)p.o + (((long)t0 + (long)ic * C) * H + h) * DV + vb, (long)H * DV, nv_of(ic), mine, w, lane);
                wave_exchange();
            }
            fresh();
            stash(nx, ic + 1);
            fresh();
            if (SETS == 1) fetch(nx, ic + 2);
            lds_barrier();
        };
        for (int ic = 0;;) {
            step(r[SETS - 1], r[0], tb[1], ic);
            if (++ic >= nchunks) break;
            step(r[0], r[SETS - 1], tb[0], ic);
            if (++ic >= nchunks) break;
        }
    };
    if (wave >= NCW) {
        if (nchunks == 0) return;
        if constexpr (!kSplitHelpers<T, DK, DIR>) helper(std::true_type{}, std::true_type{});
        else if (hw < 4) helper(std::true_type{}, std::false_type{});
        else helper(std::false_type{}, std::true_type{});
        return;
    }

    // ---- chain wave: columns vb + 16 wave + (lane & 15)
    const int m = lane & 15, g = lane >> 4;
    const int col = vb + 16 * wave + m, col16 = vb / 16 + wave;
    f32x4 S[NKT];
#pragma unroll
    for (int t = 0; t < NKT; ++t) S[t] = zero4();
    if (MODE == SCAN_STATE && p.unit_state) { // start from the identity: the final state is then the segment's transition matrix
#pragma unroll
        for (int t = 0; t < NKT; ++t)
#pragma unroll
            for (int i = 0; i < 4; ++i) S[t][i] = row4<T>(t, g) + i == col ? 1.f : 0.f;
    } else if (p.S0) {
        const float *src = p.S0 + (long)chain * DK * DV + col;
#pragma unroll
        for (int t = 0; t < NKT; ++t)
#pragma unroll
            for (int i = 0; i < 4; ++i) S[t][i] = src[(long)(row4<T>(t, g) + i) * DV];
    }
    if (nchunks > 0) {
        const int kc = LdsTile<T, DK>::kc0(lane), ks = LdsTile<T, DK>::ks0(lane), cc = LdsTile<T, C>::kc0(lane), vc = LdsTile<T, BV>::ac0(lane, wave);
        constexpr int NKS = NCT * NK, NTX = NC * (NC + 1) / 2 * TPS, NKU = NKT * NC; // operands of K S, T X, K^T Ut
        constexpr int DEPTH = sizeof(T) == 4 ? 4 : 8;
        frag Sb[NK];
        auto scale = [&](int ic) __attribute__((always_inline)) { // gated: by gamma_C of chunk ic
            const float gC = reinterpret_cast<const float *>(smem + SM::oTab + (ic & 1) * SM::szTab)[C - 1];
#pragma unroll
            for (int t = 0; t < NKT; ++t) S[t] *= gC;
        };
        auto round_state = [&]() __attribute__((always_inline)) {
#pragma unroll
            for (int s = 0; s < NK; ++s) {
                Sb[s] = as_operand(S, s, T());
                if (OUT) hand(sS, wave * NK + s, lane, Sb[s]);
            }
        };
        if constexpr (!GATED) { round_state(); lds_barrier(); }
        else { // into the first chunk's coordinates; the helpers' tables of it are there after the barrier
            lds_barrier();
            scale(0);
            round_state();
            lds_barrier();
        }
        for (int ic = 0; ic < nchunks; ++ic) {
            const unsigned char *sK = smem + SM::oK + (ic & 1) * SM::szK;
            const float *tab = reinterpret_cast<const float *>(smem + SM::oTab + (ic & 1) * SM::szTab);
            const long tile = (long)(cb + ic) * H + h;
            // A: X' = K S - V, Ut = -T X'
            f32x4 x[NCT], xv[NCT], ut[NCT], nb[NCT];
            frag xb[NC], tf[NTX], ub[NC];
#pragma unroll
            for (int t = 0; t < NCT; ++t) {
                f32x4 v = widen(read_ac<T, BV>(sV, vc, t, lane, wave));
                if (GATED) v *= tab4(tab + C, row4<T>(t, g)); // the chunk runs the plain rule on v_i / gamma_i
                x[t] = kSumFirst<T> ? zero4() : v;
                if (kSumFirst<T>) xv[t] = v;
                nb[t] = tab4(tab + 2 * C, row4<T>(t, g));
            }
            if (SAVE) {
                T *to = frag_tile<T, DK>(p.Sc, tile, DV, col16);
#pragma unroll
                for (int s = 0; s < NK; ++s) store_frag<T>(to, s, Sb[s], frag_place<T, DK>(lane));
            }
            stream<NKS + NTX, DEPTH, frag>(
                [&](auto E) __attribute__((always_inline)) {
                    constexpr int e = E;
                    if constexpr (e < NKS) return read_kc<T, DK>(sK, kc, e % NCT, e / NCT);
                    else { constexpr TilePair b = lower_pair<NC, TPS>(e - NKS); return read_kc<T, C>(sT, cc, b.t, b.s); }
                },
                [&](auto E, const frag &f) __attribute__((always_inline)) {
                    constexpr int e = E;
                    if constexpr (e == NKS) {
                        if constexpr (kSumFirst<T>)
#pragma unroll
                            for (int t = 0; t < NCT; ++t) x[t] += xv[t];
#pragma unroll
                        for (int s = 0; s < NC; ++s) xb[s] = as_operand(x, s, T());
#pragma unroll
                        for (int t = 0; t < NCT; ++t) ut[t] = kSumFirst<T> ? zero4() : nb[t] * x[t]; // the diagonal of T, which the tile leaves out
                    }
                    if constexpr (e < NKS) mma16(x[e % NCT], f, Sb[e / NCT]);
                    else {
                        constexpr TilePair b = lower_pair<NC, TPS>(e - NKS);
                        mma16(ut[b.t], f, xb[b.s]);
                        if (kTwoTerms<T>) tf[e - NKS] = f;
                    }
                });
            if constexpr (kTwoTerms<T>) {
                frag xr[NC];
#pragma unroll
                for (int s = 0; s < NC; ++s) xr[s] = rest_operand(x, xb[s], s);
                second_terms(ut, tf, xr, [](auto E) { return lower_pair<NC, TPS>(E); }, std::make_integer_sequence<int, NTX>{});
            }
            if (kSumFirst<T>)
#pragma unroll
                for (int t = 0; t < NCT; ++t) ut[t] += nb[t] * x[t];
#pragma unroll
            for (int s = 0; s < NC; ++s) {
                ub[s] = as_operand(ut, s, T());
                if (OUT) hand(sU, wave * NC + s, lane, ub[s]);
            }
            lds_barrier();
            // B: S += K^T Ut
            if (SAVE) {
                T *to = frag_tile<T, C>(p.Ut, tile, DV, col16);
#pragma unroll
                for (int s = 0; s < NC; ++s) store_frag<T>(to, s, ub[s], frag_place<T, DK>(lane));
            }
            f32x4 ku[NKT];
            if constexpr (kSumFirst<T>)
#pragma unroll
                for (int t = 0; t < NKT; ++t) ku[t] = zero4();
            stream<NKU, DEPTH, frag>([&](auto E) __attribute__((always_inline)) { return read_ks<T, DK>(sK, ks, E % NKT, E / NKT); },
                                         [&](auto E, const frag &f) __attribute__((always_inline)) { mma16(kSumFirst<T> ? ku[E % NKT] : S[E % NKT], f, ub[E / NKT]); });
            if constexpr (kSumFirst<T>)
#pragma unroll
                for (int t = 0; t < NKT; ++t) S[t] += ku[t];
            if (GATED) { // from this chunk's coordinates to the state itself, then to the next chunk's (one factor at a time: their product may leave the fp32 range)
                scale(ic);
                if (ic + 1 < nchunks) scale(ic + 1);
            }
            round_state();
            lds_barrier();
        }
    }
    if ((OUT || MODE == SCAN_STATE) && p.ST) {
        float *dst = p.ST + (long)chain * DK * DV + col;
#pragma unroll
        for (int t = 0; t < NKT; ++t)
#pragma unroll
            for (int i = 0; i < 4; ++i) dst[(long)(row4<T>(t, g) + i) * DV] = S[t][i];
    }
}

// ---- reverse -----------------------------------------------------------------------------------------------------------
// The chain carries D = -dS, with dO and T negated in the LDS, so that every product adds: dUt' = -dUt = P^T (-dO) + K D,
// dV = (-T)^T dUt', D = D + Q^T (-dO) + K^T dV.
// Per chunk it leaves -dS' (dS': the gradient with respect to the state after the chunk) in the workspace and stores dV.  The row of a
// masked token (beta zero, or below kTinyBeta) is stored as dUt_i, which the chunk kernel makes G_i and beta_i G_i from.
// STATE = true: only the gradient with respect to the initial state leaves the kernel (the first pass of a backward pass
// that is split over segments of the sequence).
template <typename T, int DK, int DV, bool GATED, bool STATE, int NCW>
__device__ __forceinline__ void scan_bwd_body(const SeqMap &sm, int H, const Ptrs &p, int bid) {
    using SM = ScanSmem<T, DK, NCW>;
    using O = Op<T>;
    typedef typename O::frag frag;
    constexpr int BV = SM::BV, NV = DV / BV, TPS = O::TPS;
    constexpr int NKT = DK / 16, NK = DK / O::KS, NCT = C / 16, NC = C / O::KS;
    constexpr bool OFF = kOffloadQdO<T>;
    static_assert(!OFF || (kSplitHelpers<T, DK, DIR_BWD> && NKT <= 4), "one tile of Q^T dO per helper that moves tiles");
    constexpr int kAuxV = BV * sizeof(T) >= 128 ? kAuxOnce : kAuxKeep; // see scan_fwd_body
    // fp32: ten waves leave each one 168 registers.  With the addresses of the waves that move tiles and the chain wave's into T carried through
    // the loop, 10 to 27 of two chain waves spilled (2 or 3 of one in the passes over segments), and a step waited for them behind its stores; so
    // these are formed in every step.  8 x 1024 tokens of 32 heads of 64, reverse scan 168 -> 164 us, gated 200 -> 167, pair 288 -> 275 and 324 -> 280; all
    // addresses of a lane formed anew take 180 and 185.  One chain wave (97 us as it is, 109 so) and d_k = 32 (112 and 114) have the registers.
    constexpr bool kFreshAddresses = sizeof(T) == 4 && DK > 32 && (NCW > 1 || STATE);
    extern __shared__ __align__(16) unsigned char smem[];
    unsigned char *sQ = smem + SM::oQ, *sD = smem + SM::oV, *sT = smem + SM::oT, *sE = smem + SM::oE, *sF = smem + SM::oF, *sO = smem + SM::oO;

    int chain, vbi;
    if (!chain_of_block(bid, sm.N * H, NV, chain, vbi)) return;
    int n = chain / H;
    const int h = chain - n * H, vb = vbi * BV;
    if (sm.order) { n = sm.order[n]; chain = n * H + h; } // packed: longest sequences first
    int t0, len, cb;
    sm.seq(n, t0, len, cb);
    const int nchunks = (len + C - 1) / C;
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6), lane = threadIdx.x & 63;

    // ---- helpers.  FORMS: the rows of tile w of P^T and of P^T dO in every chunk; MOVES: K, Q, dO, T into the LDS, dV to memory
    const int hw = helper_number<T, DK, DIR_BWD, NCW>(wave);
    auto helper = [&](auto forms, auto moves) __attribute__((always_inline)) {
        constexpr bool FORMS = decltype(forms)::value, MOVES = decltype(moves)::value;
        int lane = threadIdx.x & 63, lt = 64 * (hw & 3) + lane;
        const int w = !FORMS ? hw & 3 : NCW == 1 ? (hw == 3 ? 3 : (hw + 2) % 3) : hw < 2 ? hw : 5 - hw; // (as in the forward scan)
        // (see scan_fwd_body)
        auto fresh = [&]() __attribute__((always_inline)) {
            if (DK > 128) asm volatile("" : "+v"(lt), "+v"(lane));
            else if (kFreshAddresses) asm volatile("" : "+v"(lt));
        };
        constexpr int SETS = kScanSets<T>;
        struct Set { Pieces<T, DK> q, k; Pieces<T, BV> d; float gm[Pieces<T, BV>::NIT]; } r[SETS];
        // (of T, which is needed half a step later than the rest, one chunk at d_k = 256: with two the gated scan of 64 columns spills 14
        // registers and takes 168 us for 156, the plain one 140 for 137; 16 384 tokens of 8 heads)
        constexpr int TSETS = DK > 128 ? 1 : 2;
        Pieces<T, C> rt[TSETS];
        const int kc = LdsTile<T, DK>::kc0(lane);
        TabRegs<T, GATED> tb[2];
        // (chunks are walked from the last one down; a number below zero asks for nothing)
        auto fetch = [&](Set &x, int ic) __attribute__((always_inline)) {
            const int ii = max(ic, 0), nvalid = ic < 0 ? 0 : min(C, len - ic * C);
            const long row0 = (long)t0 + (long)ii * C, tile = (long)(cb + ii) * H + h;
            if (!MOVES) return;
            x.k.template load<kAuxKeep, true>((const T *)p.k + (row0 * H + h) * DK, (long)H * DK, nvalid, lt);
            x.q.template load<kAuxKeep, true>((const T *)p.q + (row0 * H + h) * DK, (long)H * DK, nvalid, lt);
            x.d.template load<kAuxKeep, true>((const T *)p.d_o + (row0 * H + h) * DV + vb, (long)H * DV, nvalid, lt);
            if (GATED)
#pragma unroll
                for (int it = 0; it < Pieces<T, BV>::NIT; ++it) x.gm[it] = p.gam[tile * 2 * C + ((it * NTL + lt) / Pieces<T, BV>::PPR & (C - 1))];
        };
        auto fetch_t = [&](Pieces<T, C> &x, int ic) __attribute__((always_inline)) {
            if (MOVES) x.template load<kAuxKeep, true>((const T *)p.Tm + ((long)(cb + max(ic, 0)) * H + h) * C * C, C, ic < 0 ? 0 : C, lt);
        };
        auto fetch_tab = [&](TabRegs<T, GATED> &x, int ic) __attribute__((always_inline)) {
            const int ii = max(ic, 0);
            if (MOVES) x.load(p, (long)t0 + (long)ii * C, (long)(cb + ii) * H + h, H, h, min(C, len - ii * C), lt);
        };
        auto stash = [&](Set &x, int ic) __attribute__((always_inline)) {
            if (!MOVES) return;
            x.k.store(smem + SM::oK + (ic & 1) * SM::szK, lt);
            x.q.store(sQ, lt);
            if (GATED) x.d.scale(x.gm); // o_i = gamma_i o~_i, so the plain rule's output gradient is gamma_i dO_i
            x.d.template store<true>(sD, lt);
        };
        auto tab_of = [&](int ic) __attribute__((always_inline)) { return reinterpret_cast<float *>(smem + SM::oTab + (ic & 1) * SM::szTab); };
        auto store_tab = [&](const TabRegs<T, GATED> &x, int ic) __attribute__((always_inline)) { if (MOVES) x.store(tab_of(ic), p.pro, min(C, len - max(ic, 0) * C), lt); };
        auto flush = [&](int ic) __attribute__((always_inline)) { // dV of chunk ic (past the last: nothing)
            const int ii = min(ic, nchunks - 1);
            if (MOVES) tile_out<T, BV, kAuxV>((T *)p.dv + (((long)t0 + (long)ii * C) * H + h) * DV + vb, (long)H * DV, ic < nchunks ? min(C, len - ii * C) : 0, sO, lt);
        };
        const int last = nchunks - 1;
        fetch_tab(tb[0], last); fetch_tab(tb[1], last - 1);
        fetch(r[0], last);
        fetch_t(rt[0], last);
        store_tab(tb[0], last);
        stash(r[0], last);
        __builtin_amdgcn_sched_barrier(0);
        fetch_tab(tb[0], last - 2);
        fetch(r[SETS - 1], last - 1); // (not before the first chunk is there, see scan_fwd_body)
        if (TSETS == 2) fetch_t(rt[TSETS - 1], last - 1);
        lds_barrier();
        auto step = [&](Set &nx, Set &cu, Pieces<T, C> &ht, TabRegs<T, GATED> &nt, int ic) __attribute__((always_inline)) { // nx, nt: of chunk ic - 1; ht: of chunk ic
            fresh();
            if constexpr (OFF) if constexpr (MOVES && !FORMS) { // Q^T (-dO), one tile of its rows
                const int ks = LdsTile<T, DK>::ks0(lane);
                if (w < NKT) {
                    frag qt[NC];
#pragma unroll
                    for (int s = 0; s < NC; ++s) qt[s] = read_ks<T, DK>(sQ, ks, w, s);
#pragma unroll
                    for (int c = 0; c < NCW; ++c) {
                        f32x4 f = zero4(), ob[NC];
#pragma unroll
                        for (int s = 0; s < NC; ++s) ob[s] = read_ac<T, BV>(sD, 0, s, lane, c);
#pragma unroll
                        for (int s = 0; s < NC; ++s) mma16(f, qt[s], ob[s]);
                        hand(sF, c * NKT + w, lane, f);
                    }
                }
            }
            if (MOVES) ht.template store<true>(sT, lt);
            fetch_t(ht, ic - TSETS);
            store_tab(nt, ic - 1);
            fetch_tab(nt, ic - 3);
            if (SETS == 2) fetch(cu, ic - 2); // (here rather than in B, where the LDS takes the next chunk)
            if (!STATE) flush(ic + 1);
            // for every chain wave: P^T (-dO), rows of tile t, as far as the blocks go
            auto rows_of = [&](int t, int blocks) __attribute__((always_inline)) {
                const unsigned char *own_rows = smem + SM::oK + (ic & 1) * SM::szK + (TPS == 2 ? 32 * (t >> 1) + 4 * (t & 1) : 16 * t) * LdsTile<T, DK>::RB;
                frag own[NK], pb[NC];
#pragma unroll
                for (int s = 0; s < NK; ++s) own[s] = *reinterpret_cast<const frag *>(own_rows + (kc ^ (s << 6)));
                form_p<T, DK, true>(pb, own, sQ, t, blocks, lane);
#pragma unroll
                for (int c = 0; c < NCW; ++c) {
                    f32x4 e = zero4();
                    const int vc = LdsTile<T, BV>::ac0(lane, c);
                    decltype(read_ac<T, BV>(sD, 0, 0, 0, 0)) dr[NCT];
#pragma unroll
                    for (int u = 0; u < NCT; ++u) dr[u] = read_ac<T, BV>(sD, vc, u, lane, c);
#pragma unroll
                    for (int s = 0; s < NC; ++s) if ((blocks >> s) & 1) mma16(e, pb[s], join(dr, s));
                    hand(sE, c * NCT + t, lane, e);
                }
            };
            if constexpr (FORMS) {
                const int all = ((1 << NC) - 1) & ~((1 << w / TPS) - 1);
                rows_of(w, all);
            }
            lds_barrier();
            fresh();
            stash(nx, ic - 1);
            fresh();
            if (SETS == 1) fetch(nx, ic - 2);
            lds_barrier();
        };
        for (int ic = last;;) {
            step(r[SETS - 1], r[0], rt[0], tb[1], ic);
            if (--ic < 0) break;
            step(r[0], r[SETS - 1], rt[TSETS - 1], tb[0], ic);
            if (--ic < 0) break;
        }
        if (!STATE) flush(0);
    };
    if (wave >= NCW) {
        if (nchunks == 0) return;
        if constexpr (!kSplitHelpers<T, DK, DIR_BWD>) helper(std::true_type{}, std::true_type{});
        else if (hw < 4) helper(std::true_type{}, std::false_type{});
        else helper(std::false_type{}, std::true_type{});
        return;
    }

    // ---- chain wave
    const int m = lane & 15, g = lane >> 4;
    const int col = vb + 16 * wave + m, col16 = vb / 16 + wave;
    f32x4 D[NKT]; // -dS
#pragma unroll
    for (int t = 0; t < NKT; ++t) D[t] = zero4();
    if (p.dST) {
        const float *src = p.dST + (long)chain * DK * DV + col;
#pragma unroll
        for (int t = 0; t < NKT; ++t)
#pragma unroll
            for (int i = 0; i < 4; ++i) D[t][i] = 0.f - src[(long)(row4<T>(t, g) + i) * DV];
    }
    if (nchunks > 0) {
        const int kc = LdsTile<T, DK>::kc0(lane), ks = LdsTile<T, DK>::ks0(lane), vc = LdsTile<T, BV>::ac0(lane, wave);
        int cs = LdsTile<T, C>::ks0(lane);
        const int last = nchunks - 1;
        frag Db[NK];
        lds_barrier();
        if (GATED) { // the state after the chunk is gamma_C times the plain rule's: its gradient is scaled by gamma_C on entry
            const float gC = reinterpret_cast<const float *>(smem + SM::oTab + (last & 1) * SM::szTab)[C - 1];
#pragma unroll
            for (int t = 0; t < NKT; ++t) D[t] *= gC;
        }
#pragma unroll
        for (int s = 0; s < NK; ++s) Db[s] = as_operand(D, s, T());
        constexpr int NKS = NCT * NK, NKU = NKT * NC, NTX = NC * (NC + 1) / 2 * TPS;
        constexpr int DEPTH = sizeof(T) == 4 ? 4 : 6;
        for (int ic = last; ic >= 0; --ic) {
            const unsigned char *sK = smem + SM::oK + (ic & 1) * SM::szK;
            const float *tab = reinterpret_cast<const float *>(smem + SM::oTab + (ic & 1) * SM::szTab);
            const long tile = (long)(cb + ic) * H + h;
            if (kFreshAddresses) asm volatile("" : "+v"(cs));
            // A: dUt' = K D (for now), D += Q^T (-dO) (in fp32 a helper forms that product and B adds it)
            f32x4 du[NCT];
            decltype(read_ac<T, BV>(sD, 0, 0, 0, 0)) dr[NCT];
            frag ob[NC];
#pragma unroll
            for (int t = 0; t < NCT; ++t) {
                du[t] = zero4();
                if (!OFF) dr[t] = read_ac<T, BV>(sD, vc, t, lane, wave);
            }
            if (!STATE) {
                T *to = frag_tile<T, DK>(p.dSc, tile, DV, col16);
#pragma unroll
                for (int s = 0; s < NK; ++s) store_frag<T>(to, s, Db[s], frag_place<T, DK>(lane));
            }
#pragma unroll
            for (int s = 0; s < NC; ++s) if (!OFF) ob[s] = join(dr, s);
            stream<NKS + (OFF ? 0 : NKU), DEPTH, frag>(
                [&](auto E) __attribute__((always_inline)) {
                    constexpr int e = E;
                    if constexpr (e < NKS) return read_kc<T, DK>(sK, kc, e % NCT, e / NCT);
                    else return read_ks<T, DK>(sQ, ks, (e - NKS) % NKT, (e - NKS) / NKT);
                },
                [&](auto E, const frag &f) __attribute__((always_inline)) {
                    constexpr int e = E;
                    if constexpr (e < NKS) mma16(du[e % NCT], f, Db[e / NCT]);
                    else mma16(D[(e - NKS) % NKT], f, ob[(e - NKS) / NKT]);
                });
            lds_barrier();
            // B: dUt' += P^T (-dO), dV = (-T)^T dUt', D += K^T dV (fp32: and Q^T (-dO))
            f32x4 dv[NCT], kd[NKT];
            frag db[NC], tf[NTX], nb[NC], vo[NC];
#pragma unroll
            for (int t = 0; t < NCT; ++t) {
                du[t] += take<f32x4>(sE, wave * NCT + t, lane);
                dv[t] = kSumFirst<T> ? zero4() : tab4(tab + 2 * C, row4<T>(t, g)) * du[t]; // the diagonal of T, which the tile leaves out
            }
#pragma unroll
            for (int s = 0; s < NC; ++s) db[s] = as_operand(du, s, T());
            if constexpr (kSumFirst<T>)
#pragma unroll
                for (int t = 0; t < NKT; ++t) kd[t] = zero4();
            // (of no use to the prologue variant, see dn_chunk_local.hpp)
            const bool masked = !STATE && !p.pro && __ballot(fabsf(tab[2 * C + lane]) < kTinyBeta && lane < len - ic * C) != 0;
            stream<NTX + NKU, DEPTH, frag>(
                [&](auto E) __attribute__((always_inline)) {
                    constexpr int e = E, ku = e - NTX;
                    if constexpr (ku < 0) { constexpr TilePair b = upper_pair<TPS>(kSumFirst<T> ? NTX - 1 - e : e); return read_ks<T, C>(sT, cs, b.t, b.s); }
                    else return read_ks<T, DK>(sK, ks, ku % NKT, ku / NKT);
                },
                [&](auto E, const frag &f) __attribute__((always_inline)) {
                    constexpr int e = E, ku = e - NTX;
                    if constexpr (ku == 0) {
                        if constexpr (kTwoTerms<T>) {
                            frag dr[NC];
#pragma unroll
                            for (int c = 0; c < NC; ++c) dr[c] = rest_operand(du, db[c], c);
                            second_terms(dv, tf, dr, [](auto E) { return upper_pair<TPS>(E); }, std::make_integer_sequence<int, NTX>{});
                        }
                        if (kSumFirst<T>)
#pragma unroll
                            for (int c = 0; c < NCT; ++c) dv[c] += tab4(tab + 2 * C, row4<T>(c, g)) * du[c];
#pragma unroll
                        for (int c = 0; c < NC; ++c) nb[c] = as_operand(dv, c, T());
                        if (!STATE) { // what is stored
                            if (masked)
#pragma unroll
                                for (int c = 0; c < NCT; ++c) {
                                    const f32x4 b = tab4(tab + 2 * C, row4<T>(c, g));
#pragma unroll
                                    for (int i = 0; i < 4; ++i) dv[c][i] = fabsf(b[i]) < kTinyBeta ? 0.f - du[c][i] : dv[c][i];
                                }
                            if (GATED)
#pragma unroll
                                for (int c = 0; c < NCT; ++c) dv[c] *= tab4(tab + C, row4<T>(c, g)); // v_i = gamma_i v~_i
#pragma unroll
                            for (int c = 0; c < NC; ++c) vo[c] = GATED || masked ? as_operand(dv, c, T()) : nb[c];
                        }
                    }
                    if constexpr (ku < 0) {
                        constexpr TilePair b = upper_pair<TPS>(kSumFirst<T> ? NTX - 1 - e : e);
                        mma16(dv[b.t], f, db[b.s]);
                        if (kTwoTerms<T>) tf[e] = f;
                    } else mma16(kSumFirst<T> ? kd[ku % NKT] : D[ku % NKT], f, nb[ku / NKT]);
                });
            if constexpr (kSumFirst<T>)
#pragma unroll
                for (int t = 0; t < NKT; ++t) { // (one term at a time, see kSumFirst)
                    D[t] += kd[t];
                    if (OFF) D[t] += take<f32x4>(sF, wave * NKT + t, lane);
                }
            const float gC = GATED ? tab[C - 1] : 1.f;
            if (GATED) { // across the boundary: out of this chunk's coordinates, into those of the chunk before (one factor at a time: their product may leave the fp32 range)
#pragma unroll
                for (int t = 0; t < NKT; ++t) D[t] *= gC;
                if (ic > 0) {
                    const float gN = reinterpret_cast<const float *>(smem + SM::oTab + ((ic - 1) & 1) * SM::szTab)[C - 1];
#pragma unroll
                    for (int t = 0; t < NKT; ++t) D[t] *= gN;
                }
            }
#pragma unroll
            for (int s = 0; s < NK; ++s) Db[s] = as_operand(D, s, T());
            if (!STATE) {
#pragma unroll
                for (int t = 0; t < NCT; ++t)
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        const int byte = (16 * wave + m) * (int)sizeof(T);
                        *reinterpret_cast<T *>(sO + LdsTile<T, BV>::at(row4<T>(t, g) + i, byte >> 4) + (byte & 15)) = vo[t / TPS][4 * (t % TPS) + i];
                    }
            }
            lds_barrier();
        }
    }
    if (p.dS0) {
        float *dst = p.dS0 + (long)chain * DK * DV + col;
#pragma unroll
        for (int t = 0; t < NKT; ++t)
#pragma unroll
            for (int i = 0; i < 4; ++i) dst[(long)(row4<T>(t, g) + i) * DV] = 0.f - D[t][i];
    }
}

} // namespace dn
