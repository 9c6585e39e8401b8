// The chunk-parallel backward kernel in bf16: everything of the backward pass that is local to one chunk, given the chunk-initial
// state S, the gradient dS' with respect to the state after the chunk, Ut (Eq. 8) and dV from the two scans.
//
// Inside a chunk Ut solves (I + A) Ut = diag(beta) (V - K S) with A = diag(beta) tril(K K^T, -1) (Eq. 10-11), so with dUt =
// P^T dO + K dS' the adjoint of the solve is G = (I + A)^-T dUt, and everything follows from G and Ut:
//     dV = diag(beta) G  (that is T^T dUt: the reverse scan forms it and stores it),    dA = -tril(G Ut^T, -1).
// The inverse of Eq. 10 and the gradients with respect to W and T never have to exist here.  Per chunk:
//     dP = tril(dO Ut^T)                  Ah = diag(beta) dA = -tril(dV Ut^T, -1)
//     dQ = dO S^T + dP K                  dK = Ut dS'^T - dV S^T + dP^T Q + (Ah + Ah^T) K
//     dbeta_i = G_i . (v_i - S_{i-1}^T k_i) = (dV_i . v_i - (dV S^T)_i . k_i + sum_{j<i} (k_i . k_j) Ah_ij) / beta_i
// The second term takes dV S^T, which dK needs anyway, from the fp32 accumulators, so K S is never formed; the third takes Ah and
// K K^T from theirs.  In dbeta only dV carries a rounding of the row itself.  (The shorter form dV_i . Ut_i / beta_i^2, the diagonal of
// dV Ut^T, has Ut_i's as well: 12 to 22 % further from the exact dbeta, 30 % in the gated variant.)
// Where beta is zero (a masked token), or so small that the quotient could leave the range of the types, the reverse scan has
// left dUt_i in the place of dV_i, and dbeta_i = G_i . e_i with G_i = dUt_i - sum_{j>i} (k_i . k_j) dV_j and e_i = v_i - S^T k_i -
// sum_{j<i} (k_i . k_j) Ut_j; see masked_rows.  (The prologue variant needs none of it: its gradient is that of the logit,
// dlogit_i = beta_i (1 - beta_i) G_i . e_i, which has no quotient.)
// Gated rule: the chunk is the plain rule on v_i / gamma_i with outputs gamma_i o~_i, so rows of dO and dV count gamma_i times.  The
// tiles stay as they are and the rows of the products are scaled, in fp32, but for strongly decaying chunks (see `strong`).
//
// What bounds it and why it is cut as it is.  A tile is 160 KB in and 32 KB out at d = 128: 818 MB of counted traffic for 4096 of them (16 384 tokens of
// 16 heads), 134 us at the 6.1 TB/s of a large copy.  The form that holds the tiles on their way in registers (dn_chunk_local.hpp) takes 161 us there, 131 of
// them also when every tile is found in the L2: 19 K cycles a tile, 5.3 K of them moving registers to the LDS while the matrix cores wait, 3.8 K in K K^T
// and the triangles on three of eight waves.  Here the tiles travel straight to the LDS (no registers, no moves, one barrier interval per block instead
// of two), an operand of a C x d_k product serves both token blocks, K S is not formed, and the results leave four or eight at a time.  Between event
// records, the form through registers and this one, us, 16 384 tokens of width 2048: d = 128 163 -> 138, gated 214 -> 157, prologue 214 -> 173, d = 64 131 -> 115,
// its prologue 168 -> 147; of 16 heads of 128 x 64 116 -> 103; of 32 heads of 64 x 128 215 -> 176; 5 x 1500 tokens of d = 128 85 -> 70, 32 768 tokens 311 -> 267.
// A tenth of the tokens masked: d = 128 189 -> 168, gated 246 -> 205, d = 64 160 -> 130, 128 x 64 131 -> 127, 64 x 128 274 -> 236.
// With the second block of a chunk requested at the start of the chunk, not when the chunk before it is done with its own, d = 128, gated and prologue
// took 147, 166 and 174 for 138, 153 and 172.
#pragma once
#include <type_traits>

#include "dn_kernels.hpp"

namespace dn {

// ---- tiles in the LDS --------------------------------------------------------------------------------------------------
// Rows of COLS elements without padding; the 16-byte pieces of a row are permuted by an XOR with a function of the row, chosen so that
// both kinds of operand read of the 32 x 32 x 16 products (one piece of 32 rows; for the transposing read four pieces of four
// rows) spread over all 64 banks.
template <int COLS> struct RowTile {
    static constexpr int RB = 2 * COLS, PPR = RB / 16, bytes = C * RB;
    __device__ static int swz(int r) {
        if (PPR >= 16) return ((r & 3) << 2) | ((r >> 2) & 3);
        if (PPR == 8) return ((r & 2) << 1) | ((r >> 2) & 3);
        return (r >> 2) & 3;
    }
    __device__ static int at(int r, int piece) { return r * RB + ((piece ^ swz(r)) << 4); }
    // operand with the contraction index along the rows: row n0 + (l & 31), indices 16 s + 8 (l >> 5) + 0 .. 7
    __device__ static int kc0(int lane) { return at(lane & 31, lane >> 5); }
    __device__ static int kc(int kc0, int n0, int s) { return (kc0 ^ (s << 5)) + n0 * RB; }
    // ... across the rows: column n0 + (l & 31), rows k0 + 8 (l >> 5) + 0 .. 7, as two reads (the second at ks_hi)
    __device__ static int ks_lo(int lane, int n0) {
        const int i = lane & 15;
        return at(8 * (lane >> 5) + (i >> 2), (n0 >> 3) + 2 * ((lane >> 4) & 1) + ((i & 3) >> 1)) + 8 * (i & 1);
    }
    __device__ static int ks_hi(int lo) { return (lo ^ 16) + 4 * RB; }
};
// The tiles that the scans left in the order of their operands (store_frag): blocks of 16 state columns x 32 entries (of d_k, or
// tokens), a kilobyte each; entries 8 g .. 8 g + 7 of column v are piece 16 g + (v ^ 4 g).  Operand with the contraction index
// across the columns: entry l & 31 of the block, columns 8 (l >> 5) + 0 .. 7
__device__ inline int frag_ks_lo(int lane) {
    const int i = lane & 15, g = 2 * ((lane >> 4) & 1) + ((i & 3) >> 1), v = 8 * (lane >> 5) + (i >> 2);
    return 256 * g + ((v ^ (4 * g)) << 4) + 8 * (i & 1);
}
// ... along the entries: column l & 31 (two blocks, ROWS / 32 kilobytes apart), entries 16 s + 8 (l >> 5) + 0 .. 7
template <int ROWS> __device__ inline int frag_kc(int lane, int s) {
    const int v = lane & 15, g = 2 * (s & 1) + (lane >> 5);
    return ((lane >> 4) & 1) * (ROWS / 32) * 1024 + (s >> 1) * 1024 + 256 * g + ((v ^ (4 * g)) << 4);
}
__device__ inline bf16x8 lds16(const unsigned char *p) { return *reinterpret_cast<const bf16x8 *>(p); }
__device__ inline bf16x8 lds_tr16(const unsigned char *lo, const unsigned char *hi) {
    return __builtin_bit_cast(bf16x8, __builtin_shufflevector(lds_tr(lo), lds_tr(hi), 0, 1, 2, 3, 4, 5, 6, 7));
}
// 64 lanes' 16 bytes from global memory to a kilobyte of the LDS, without registers in between (M0 holds the place, lane l lands 16 l
// behind it; lanes past the descriptor's range leave zeros).  The compiler does not know of the transfer: wait_dma before the
// barrier that makes the data readable.
// The hardware does not hold back a buffer access that reads a scalar register written on the vector unit (readlane, readfirstlane: so come
// spilled descriptors and offsets back) fewer than five wait states before, and the compiler, which keeps that distance for its own accesses, does not
// look into an asm: the move and the s_nop are five by themselves (M0 needs one), whatever stands ahead of them.  The compiler does not know that M0 is
// written either: nothing else in a kernel with these transfers may use it.  tests/test_dma_hazards_host.py reads both from the compiled code.
__device__ __forceinline__ void dma16(__amdgpu_buffer_rsrc_t rs, int voff, int soff, unsigned lds) {
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 3\n\tbuffer_load_dwordx4 %1, %2, %3 offen nt lds" ::"s"(lds), "v"(voff), "s"(rs), "s"(soff) : "memory");
}
// N: how many requests this wave has certainly made after the transfers it waits for
template <int N> __device__ __forceinline__ void wait_dma() { asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory"); }
__device__ inline unsigned lds_offset(const unsigned char *p) {
    typedef __attribute__((address_space(3))) const unsigned char lds_t;
    return (unsigned)(size_t)(lds_t *)p;
}
// Eight neighbouring rows of this lane's column of an accumulator, 16 g + 8 (l >> 5) .., as bf16: a lane holds four of every eight, the lane
// across the other four
__device__ inline uint4 row8(const f32x16 &o, int g) {
    typedef unsigned u32x2 __attribute__((ext_vector_type(2)));
    const u32x2 a = __builtin_bit_cast(u32x2, bf16x4{(bf16)o[8 * g], (bf16)o[8 * g + 1], (bf16)o[8 * g + 2], (bf16)o[8 * g + 3]});
    const u32x2 b = __builtin_bit_cast(u32x2, bf16x4{(bf16)o[8 * g + 4], (bf16)o[8 * g + 5], (bf16)o[8 * g + 6], (bf16)o[8 * g + 7]});
    const auto x = __builtin_amdgcn_permlane32_swap(a[0], b[0], false, false), y = __builtin_amdgcn_permlane32_swap(a[1], b[1], false, false);
    return make_uint4(x[0], y[0], x[1], y[1]);
}
// sum of the products of two times eight elements, added to s (fp32 accumulation)
__device__ inline float dot8(const uint4 &a, const uint4 &b, float s) {
    typedef bf16 bf16x2 __attribute__((ext_vector_type(2)));
    const unsigned x[4] = {a.x, a.y, a.z, a.w}, y[4] = {b.x, b.y, b.z, b.w};
#pragma unroll
    for (int i = 0; i < 4; ++i) s = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, x[i]), __builtin_bit_cast(bf16x2, y[i]), s, false);
    return s;
}

// Gradient through the feature map of section 3.3 for eight neighbouring elements x of a row that LANES lanes hold: with y = SiLU(x) / n,
// n = ||SiLU(x)||,   dx = SiLU'(x) (dy - y (y . dy)) / n,   SiLU'(x) = s + x s (1 - s), in this order: s + x s - x s^2 loses the one next to a large x.
// The norm and y . dy are summed in one pass (the fast sigmoid: y need not have the bits of the mapped tile here).
template <int LANES> __device__ __forceinline__ u32x4 map_gradient(const uint4 &xr, const u32x4 &dyr) {
    const bf16x8 x = __builtin_bit_cast(bf16x8, xr), dy = __builtin_bit_cast(bf16x8, dyr);
    float sg[8], sv[8], ss = 0.f, d = 0.f;
#pragma unroll
    for (int u = 0; u < 8; ++u) {
        const float xv = (float)x[u];
        sg[u] = sigmoid_fast_f32(xv);
        sv[u] = xv * sg[u];
        ss = __fmaf_rn(sv[u], sv[u], ss);
        d = __fmaf_rn(sv[u], (float)dy[u], d);
    }
    ss = lane_sum<LANES>(ss);
    d = lane_sum<LANES>(d);
    const float inv = ss > 0.f ? __frsqrt_rn(ss) : 0.f, t = (d * inv) * inv; // (a row whose image is exactly zero has no gradient)
    bf16x8 o;
#pragma unroll
    for (int u = 0; u < 8; ++u) o[u] = (bf16)(__fmaf_rn(-sv[u], t, (float)dy[u]) * (__fmaf_rn(sv[u], 1.f - sg[u], sg[u]) * inv));
    return __builtin_bit_cast(u32x4, o);
}

struct NoPieces {};

template <int DK, int DV> struct ChunkSmem {
    static constexpr int BVB = 64, NB = DV / BVB; // state columns per block, blocks per chunk
    using KT = RowTile<DK>;
    using VT = RowTile<BVB>;
    using PT = RowTile<32>;
    static constexpr size_t szPT = 32 * PT::RB; // a 32 x 32 tile of dP or Ah
    static constexpr size_t oK = 0, oQ = oK + KT::bytes, oB = oQ + KT::bytes;
    // a block: S, -dS', dO, dV, Ut
    static constexpr size_t szS = (size_t)BVB * DK * 2, szU = (size_t)BVB * C * 2;
    static constexpr size_t bS = 0, bDS = bS + szS, bDO = bDS + szS, bDV = bDO + VT::bytes, bUt = bDV + VT::bytes, szB = bUt + szU;
    // two blocks, one worked on and one on its way (where that holds: see settle); at 64 x 64 one, and two workgroups per CU that work while the other one waits
    static constexpr int NBUF = DK == 64 && DV == 64 ? 1 : 2;
    static constexpr size_t oTab = oB + NBUF * szB;
    static constexpr size_t oBeta = oTab, oGam = oBeta + 4 * C, oCv = oGam + 4 * C, oPl = oCv + 4 * C; // v_i . dv_i;  third term of dbeta, per 32 tokens j
    static constexpr size_t oPr = oPl + 4 * 2 * C;  // second term of dbeta per wave that holds rows of dK
    static constexpr size_t oCq = oPr + 4 * 4 * C;  // gated: q_i . dq_i per wave that holds rows of dQ
    static constexpr size_t oPm = oCq + 4 * 4 * C;  // dbeta of the masked rows, per 32 columns of a block
    static constexpr size_t oZ = oPm + 4 * 2 * C;   // gated: per-wave shares of <dS_C, S_C> and <dS_0, S_0>
    static constexpr size_t endTab = oZ + 4 * 2 * NWC;
    static constexpr size_t oP = endTab, oA = oP + 3 * szPT; // dP and Ah, three 32 x 32 tiles each
    static constexpr size_t oMV = endTab;                    // ... and, while a block is worked on, V of the masked rows
    static constexpr size_t bytes = endTab + cmax(VT::bytes, 6 * szPT);
    static_assert(DK <= 128 && (NB == 1 || (NB == 2 && NBUF == 2)), "a chunk's blocks alternate between the two buffers");
    static constexpr int WPC = bytes <= 80 * 1024 ? 2 : 1; // workgroups per CU
};

// Work is split by result: waves 0 .. 3 form dQ and (a 32 x 32 tile each) dP and Ah, waves 4 .. 7 form dK; a wave owns 32 columns of
// d_k and RB blocks of 32 tokens of its matrix (d_k = 128: both, so that an operand that runs over columns serves two products).  All products
// are formed transposed, d_k (or the token j) in the accumulator's rows and the token in the lane: a row sum is then one over a wave's own registers,
// and four neighbouring elements of a row leave in one piece.
template <int DK, int DV, int VAR>
__device__ __forceinline__ void bwd_local_bf16(SeqMap sm, int H, Ptrs p, int chunks_total) {
    using SM = ChunkSmem<DK, DV>;
    using KT = typename SM::KT;
    using VT = typename SM::VT;
    using PT = typename SM::PT;
    constexpr bool GATED = VAR == VAR_GATED, PRO = VAR == VAR_PROLOGUE;
    constexpr int BVB = SM::BVB, NB = SM::NB, KSB = BVB / 16;
    constexpr int RB = DK == 128 ? 2 : 1;
    constexpr int NKW = RB == 2 ? 4 : 2; // waves that share a row of dQ (dK)
    constexpr int NST = 2 * (C * KT::PPR / NTC); // output stores of a thread
    extern __shared__ __align__(16) unsigned char smem[];
    unsigned char *sK = smem + SM::oK, *sQ = smem + SM::oQ, *sP = smem + SM::oP, *sA = smem + SM::oA;
    float *sBeta = reinterpret_cast<float *>(smem + SM::oBeta), *sGam = reinterpret_cast<float *>(smem + SM::oGam);
    float *sCv = reinterpret_cast<float *>(smem + SM::oCv), *sPl = reinterpret_cast<float *>(smem + SM::oPl), *sPr = reinterpret_cast<float *>(smem + SM::oPr);
    float *sCq = reinterpret_cast<float *>(smem + SM::oCq), *sPm = reinterpret_cast<float *>(smem + SM::oPm), *sZ = reinterpret_cast<float *>(smem + SM::oZ);
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);

    auto run = [&](auto dk_role) __attribute__((always_inline)) {
        constexpr bool DKW = decltype(dk_role)::value;
        const int w4 = wave & 3;
        // The thread index, re-read through an empty asm in every barrier interval: the per-lane addresses derived from it are then formed
        // where they are used instead of being carried through the whole tile loop.
        unsigned tid = threadIdx.x; int lane = tid & 63, hh = lane >> 5, li = lane & 31;
        auto fresh = [&]() __attribute__((always_inline)) {
            tid = threadIdx.x;
            asm volatile("" : "+v"(tid));
            lane = tid & 63; hh = lane >> 5; li = lane & 31;
        };
        // column block kb; token blocks r ^ ti; the tile (token block ti, token block tj) of dP and Ah
        const int kb = RB == 2 ? w4 : w4 & 1, ti = DKW && RB == 2 ? 0 : w4 >> 1, tj = w4 & 1;
        // columns 32 kb + 8 g + 4 hh .. (four of them) of row 32 r + li in K or Q
        auto row4k = [&](const unsigned char *t, int r, int g) __attribute__((always_inline)) {
            return widen(*reinterpret_cast<const s16x4 *>(t + (32 * r + li) * KT::RB + (((4 * kb + g) ^ KT::swz(li)) << 4) + 8 * hh));
        };

        // ---- requests
        struct Head {
            TileRegs<bf16, C, DK, NTC> k, q;
            unsigned beta; // the bits of one element
            float gm;
        } rh;
        std::conditional_t<PRO, TileRegs<bf16, C, DK, NTC>, NoPieces> rawq, rawk;
        uint4 rv[2] = {make_uint4(0, 0, 0, 0), make_uint4(0, 0, 0, 0)}; // V: of a chunk's first block, of the others
        static_assert(NTC == C * VT::PPR, "one piece of a C x BVB tile per thread");
        auto vr = [&]() __attribute__((always_inline)) { return tid / VT::PPR; };
        auto vp = [&]() __attribute__((always_inline)) { return tid % VT::PPR; };
        const unsigned lds0 = __builtin_amdgcn_readfirstlane(lds_offset(smem) + 1024 * wave);
        constexpr int NS = (int)(SM::szS / 8192), NDMA = 2 * NS + 3; // a wave's transfers of S, and per block
        static_assert(SM::szS % 8192 == 0 && VT::bytes == 8192 && SM::szU == 8192, "whole rounds");
        auto fetch_blk = [&](const TilePos &tp, int vb, int buf) __attribute__((always_inline)) {
            const unsigned to = lds0 + (unsigned)(SM::oB + buf * SM::szB);
            const long tv = tp.tile * DV + vb * BVB;
            const __amdgpu_buffer_rsrc_t rs = make_rsrc((const bf16 *)p.Sc + tv * DK), rd = make_rsrc((const bf16 *)p.dSc + tv * DK), ru = make_rsrc((const bf16 *)p.Ut + tv * C);
            const long row = (tp.row0 * H + tp.h) * DV + vb * BVB;
            const int stride = H * DV * 2;
            const __amdgpu_buffer_rsrc_t ro = make_rsrc((const bf16 *)p.d_o + row, tp.nvalid * stride), rw = make_rsrc((const bf16 *)p.dv + row, tp.nvalid * stride);
#pragma unroll
            for (int j = 0; j < NS; ++j) {
                dma16(rs, 16 * lane, 8192 * j + 1024 * wave, to + (unsigned)SM::bS + 8192 * j);
                dma16(rd, 16 * lane, 8192 * j + 1024 * wave, to + (unsigned)SM::bDS + 8192 * j);
            }
            constexpr int RPW = 64 / VT::PPR; // rows of a kilobyte
            const int vsrc = ((lane % VT::PPR) ^ VT::swz(RPW * wave + lane / VT::PPR)) * 16; // the piece that lands in this lane's place
            const int voff = (RPW * wave + lane / VT::PPR) * stride + vsrc;
            dma16(ro, voff, 0, to + (unsigned)SM::bDO);
            dma16(rw, voff, 0, to + (unsigned)SM::bDV);
            dma16(ru, 16 * lane, 1024 * wave, to + (unsigned)SM::bUt);
        };
        auto v_of = [&](int vb) __attribute__((always_inline)) {
            const uint4 a = rv[0], b = rv[1];
            return vb > 0 ? b : a;
        };
        auto fetch_v = [&](uint4 &x, const TilePos &tp, int vb, int live) __attribute__((always_inline)) {
            const __amdgpu_buffer_rsrc_t rs = make_rsrc((const bf16 *)p.v + (tp.row0 * H + tp.h) * DV + vb * BVB, tp.nvalid * live * H * DV * 2);
            x = buf_load16<kAuxOnce>(rs, vr() * H * DV * 2 + 16 * vp(), 0);
        };
        auto fetch_head = [&](const TilePos &tp, int live) __attribute__((always_inline)) {
            // (prologue variant: the q and k that k_wy_prep mapped and left in the workspace, in the layout of q and k)
            rh.k.load_once((const bf16 *)(PRO ? p.Km : p.k) + (tp.row0 * H + tp.h) * DK, (long)H * DK, tp.nvalid * live, tid);
            rh.q.load_once((const bf16 *)(PRO ? p.Qm : p.q) + (tp.row0 * H + tp.h) * DK, (long)H * DK, tp.nvalid * live, tid);
            rh.beta = ((const unsigned short *)p.beta)[(tp.row0 + min(lane, tp.nvalid - 1)) * H + tp.h]; // (every wave: each looks for masked rows)
            if (GATED) rh.gm = p.gam[tp.tile * 2 * C + lane];
        };
        // The compiler does not know of the transfers, and takes a wait for a register load that was made before some of them for one that lets only
        // later loads and stores be under way: it would wait for the transfers too.  So the registers loaded in a chunk's first block are marked as
        // written in its second one, before that requests anything.  Not covered: the position of the next tile (in the loop its loads go through the vector
        // memory, and where the paths of the two layouts meet the compiler waits for everything), the first use of K and Q in a chunk, and with one
        // block per chunk V.  As compiled each of them waits for all that is under way, so a chunk begins with nothing on its way.
        auto settle = [&](uint4 &x) __attribute__((always_inline)) { asm volatile("" : "+v"(x.x), "+v"(x.y), "+v"(x.z), "+v"(x.w)); };
        auto settle_all = [&]() __attribute__((always_inline)) {
            settle(rv[0]); settle(rv[1]);
#pragma unroll
            for (int i = 0; i < TileRegs<bf16, C, DK, NTC>::NIT; ++i) {
                settle(rh.k.v[i]); settle(rh.q.v[i]);
                if constexpr (PRO) { settle(rawq.v[i]); settle(rawk.v[i]); }
            }
            asm volatile("" : "+v"(rh.beta));
            if (GATED) asm volatile("" : "+v"(rh.gm));
        };
        auto pos_of = [&](const TileIter &it) __attribute__((always_inline)) {
            TilePos tp{0, 0, 0, 0, false};
            if (it.valid()) tp = tile_pos(sm, H, it.gid(), it.head());
            // (the same in every lane, in scalar registers; rows and tiles are counted in 31 bits)
            auto uni = [](int x) { return __builtin_amdgcn_readfirstlane(x); };
            return TilePos{uni(tp.nvalid), uni(tp.h), uni((int)tp.row0), uni((int)tp.tile), uni(tp.ok) != 0};
        };

        TileIter it(chunks_total, H);
        TilePos cur = pos_of(it);
        int par = 0; // the buffer of the chunk's first block (one block per chunk: they alternate)
        if (cur.ok) {
            fetch_head(cur, 1);
            fetch_v(rv[0], cur, 0, 1);
            fetch_blk(cur, 0, 0);
            if (NB > 1) fetch_blk(cur, 1, 1);
            wait_dma<0>();
        }
        while (cur.ok) { // packed layout: the first chunk past the last real one ends the walk (so would every later one)
            TileIter nx = it;
            nx.next();
            const TilePos np = pos_of(nx);
            const TilePos nf = np.ok ? np : cur; // what the freed registers request at the end (masked where there is no next chunk)
            const int nl = np.ok ? 1 : 0;
            const int nvalid = cur.nvalid, h = cur.h;
            const long row0 = cur.row0;

            auto put = [&](const TileRegs<bf16, C, DK, NTC> &x, unsigned char *t) __attribute__((always_inline)) {
#pragma unroll
                for (int i = 0; i < TileRegs<bf16, C, DK, NTC>::NIT; ++i)
                    *reinterpret_cast<uint4 *>(t + KT::at(i * (NTC / KT::PPR) + tid / KT::PPR, tid % KT::PPR)) = x.v[i];
            };
            put(rh.k, sK); put(rh.q, sQ);
            float b = lane < nvalid ? __uint_as_float(rh.beta << 16) : 0.f;
            if (PRO) b = lane < nvalid ? sigmoid_f32(b) : 0.f; // beta = sigmoid(logit), section 2.2
            const unsigned long long masked = PRO ? 0ull : __ballot(lane < nvalid && fabsf(b) < kTinyBeta); // the same in every wave
            if (!DKW && w4 == 0) {
                sBeta[lane] = b;
                if (GATED) sGam[lane] = rh.gm;
            }
            // Gated rule under strong decay: gamma runs from e^h to e^-h over the chunk (it is relative to the chunk's middle), Ut as stored from e^-h to
            // e^h, S and dS' stand at e^-h.  A product with a row that is scaled only afterwards can leave fp32 where the scaled row's would not, and where
            // scaled rows become subnormal the scans have lost what dq would still hold, which dg takes for a gradient.  So from h = 60 on the rows of dO and
            // dV are scaled in the tiles, rounded as in the scans.  (h = 78: dO ~ 1e4 overflowed, at dO ~ 1e-6 dg was off by its own size instead
            // of a tenth.  h = 51: dO from 1e-10 to 1e4 shows no difference but that of the rounding, dq 3.0e-3 off instead of 3.3e-3.)
            const bool strong = GATED && __builtin_amdgcn_readlane(__float_as_uint(GATED ? rh.gm : 0.f), C - 1) < (int)__float_as_uint(0x1p-87f);
            auto gamma = [&](int i) __attribute__((always_inline)) { return strong ? 1.f : sGam[i]; }; // what row i of a product still has to be multiplied by
            auto scale_piece = [&](unsigned char *at, float g) __attribute__((always_inline)) {
                bf16x8 t = lds16(at);
#pragma unroll
                for (int u = 0; u < 8; ++u) t[u] = (bf16)((float)t[u] * g);
                *reinterpret_cast<bf16x8 *>(at) = t;
            };

            f32x16 x[RB], y[RB], dp = zero16(), ah = zero16(); // x: dO S^T or dV S^T;  y: -Ut dS'^T
#pragma unroll
            for (int r = 0; r < RB; ++r) { x[r] = zero16(); y[r] = zero16(); }
            float cv = 0.f, zs = 0.f, pm = 0.f; // this thread's shares of v_i . dv_i, <S, dS'>, dbeta of its masked row

            // dbeta and dV of the masked rows, over the columns of block vb, by waves 0 .. 3: tile of 32 columns ub, 32 tokens ua.  In the
            // accumulators a lane has 16 columns of its token i, so each of e_i and G_i is one more product with a masked K K^T, formed once a
            // chunk in operand order, and G_i . e_i a sum over registers.  In the tile of dV the masked rows are zero meanwhile (dV_i = beta_i G_i,
            // and beta_i is zero but for the tiny ones, which are filled in at the end).  Ut_i = beta_i e_i holds for them as for any row, so
            // nothing else of the chunk is touched.
            bf16x8 le[2], lg[2], lo[2]; // tril(K K^T, -1) within the tokens' own 32: below i, above i; the other 32 tokens
            auto masked_rows = [&](const unsigned char *blk, unsigned char *sDV, int vb) __attribute__((always_inline)) {
                const int ua = w4 & 1, ub = w4 >> 1, i = 32 * ua + li;
                const bool does = !DKW && ((masked >> (32 * ua)) & 0xffffffffull), mine = does && ((masked >> i) & 1);
                unsigned char *sMV = smem + SM::oMV;
                if ((masked >> vr()) & 1) *reinterpret_cast<uint4 *>(sMV + VT::at(vr(), vp())) = v_of(vb);
                s16x4 du[4];
                if (mine)
#pragma unroll
                    for (int u = 0; u < 4; ++u) {
                        s16x4 *at = reinterpret_cast<s16x4 *>(sDV + VT::at(i, 4 * ub + u) + 8 * hh);
                        du[u] = *at;
                        *at = s16x4{0, 0, 0, 0};
                    }
                lds_barrier();
                if (does) {
                    const int kc_k = KT::kc0(lane);
                    if (vb == 0) {
                        // rows of an accumulator in the order that makes it the operand of a product over these rows
                        const int perm = 16 * (li >> 4) + 8 * ((li >> 2) & 1) + 4 * ((li >> 3) & 1) + (li & 3);
                        f32x16 near = zero16(), far = zero16();
#pragma unroll
                        for (int s = 0; s < DK / 16; ++s) {
                            const bf16x8 k = lds16(sK + KT::kc(kc_k, 32 * ua, s));
                            mfma32(near, lds16(sK + KT::at(32 * ua + perm, 2 * s + hh)), k);
                            mfma32(far, lds16(sK + KT::at(32 * (ua ^ 1) + perm, 2 * s + hh)), k);
                        }
#pragma unroll
                        for (int t = 0; t < 2; ++t) {
                            const int s = 2 * ua + t, so = 2 * (ua ^ 1) + t, below_i = li - 16 * t - 8 * hh; // token i - token j of element 0
#pragma unroll
                            for (int e = 0; e < 8; ++e) {
                                const float v = near[8 * t + e], f = far[8 * t + e];
                                le[t][e] = (bf16)(below_i > e ? v : 0.f);
                                lg[t][e] = (bf16)(below_i < e ? (GATED ? v * sGam[16 * s + 8 * hh + e] : v) : 0.f);
                                lo[t][e] = (bf16)(GATED && !ua ? f * sGam[16 * so + 8 * hh + e] : f);
                            }
                        }
                    }
                    f32x16 ks = zero16(), g = zero16(); // (K S)^T
#pragma unroll
                    for (int s = 0; s < DK / 16; ++s)
                        mfma32(ks, lds16(blk + SM::bS + 2 * ub * (DK / 32) * 1024 + frag_kc<DK>(lane, s)), lds16(sK + KT::kc(kc_k, 32 * ua, s)));
                    auto below = [&](const bf16x8 &l, int s) __attribute__((always_inline)) { // + (tril(K K^T, -1) Ut)^T over tokens 16 s ..
                        mfma32(ks, lds16(blk + SM::bUt + 2 * ub * 2 * 1024 + frag_kc<C>(lane, s)), l);
                    };
                    auto above = [&](const bf16x8 &l, int s) __attribute__((always_inline)) { // (tril(K K^T, -1)^T dV)^T
                        const int at = VT::ks_lo(lane, 32 * ub) + 16 * s * VT::RB;
                        mfma32(g, lds_tr16(sDV + at, sDV + VT::ks_hi(at)), l);
                    };
#pragma unroll
                    for (int t = 0; t < 2; ++t) {
                        below(le[t], 2 * ua + t);
                        above(lg[t], 2 * ua + t);
                        if (ua) below(lo[t], t);
                        else above(lo[t], 2 + t);
                    }
                    if (mine) {
                        const long at = ((row0 + i) * H + h) * DV + vb * BVB + 32 * ub + 4 * hh;
                        float gm = 1.f, gi = 1.f; // gated: the products are in the chunk's coordinates
                        if (GATED) { gm = sGam[i]; gi = 1.f / gm; }
                        const float bi = sBeta[i];
#pragma unroll
                        for (int u = 0; u < 4; ++u) {
                            const f32x4 d = widen(du[u]), vv = widen(*reinterpret_cast<const s16x4 *>(sMV + VT::at(i, 4 * ub + u) + 8 * hh));
                            bf16 out[4];
#pragma unroll
                            for (int e = 0; e < 4; ++e) {
                                const float gg = d[e] * gm - g[4 * u + e];
                                pm += gg * (vv[e] * gi - ks[4 * u + e]);
                                out[e] = from_f32<bf16>(gg * bi * gi);
                            }
                            st4v((bf16 *)p.dv + at + 8 * u, out);
                            s16x4 raw;
                            __builtin_memcpy(&raw, out, 8);
                            du[u] = raw;
                        }
                    }
                }
                if (__ballot(lane < nvalid && ((masked >> lane) & 1) && sBeta[lane] != 0.f)) {
                    lds_barrier();
                    if (mine)
#pragma unroll
                        for (int u = 0; u < 4; ++u) *reinterpret_cast<s16x4 *>(sDV + VT::at(i, 4 * ub + u) + 8 * hh) = du[u];
                    lds_barrier();
                } else if (strong) {
                    lds_barrier(); // (the tile is about to be scaled)
                }
                // (no barrier otherwise: waves 4 .. 7 go on with their products.  V of the masked rows is not overwritten before the next barrier)
            };

            auto block = [&](int vb) __attribute__((always_inline)) {
                const int buf = SM::NBUF == 1 ? 0 : NB == 1 ? par : vb & 1;
                unsigned char *blk = smem + SM::oB + buf * SM::szB;
                // Requests after a first block's transfers: the chunk's second block, if there is one, and the stores of the chunk before, at the least (masked
                // rows, dbeta and the gate's gradient store more).  The waits named at settle stand ahead of this one and are the ones that bind.
                if (vb > 0) wait_dma<0>();
                else wait_dma<NST + (NB > 1 ? NDMA : 0)>();
                lds_barrier(); fresh();
                if (vb > 0) settle_all();
                // every wave is done with the other buffer: the next chunk's first block travels while this one is worked on (a second block has been
                // requested when the chunk before was done with its own, and has arrived by the first block of its own chunk)
                if (vb + 1 == NB && SM::NBUF == 2 && np.ok) fetch_blk(np, 0, buf ^ 1);
                if (masked) { masked_rows(blk, blk + SM::bDV, vb); fresh(); }
                // v_i . dv_i
                cv = dot8(v_of(vb), *reinterpret_cast<const uint4 *>(blk + SM::bDV + VT::at(vr(), vp())), cv);
                if (strong) { // (a thread scales the piece that it has just taken its sum from)
                    const float g = sGam[vr()];
                    scale_piece(blk + SM::bDO + VT::at(vr(), vp()), g);
                    scale_piece(blk + SM::bDV + VT::at(vr(), vp()), g);
                    lds_barrier(); fresh();
                }
                if (vb + 1 < NB) fetch_v(rv[1], cur, vb + 1, 1);
                if (vb == 0) {
                    fetch_v(rv[0], nf, 0, nl);
                    fetch_head(nf, nl);
                    if constexpr (PRO) { // the pre-activations, for the way back through the map
                        rawq.load_once((const bf16 *)p.q + (row0 * H + h) * DK, (long)H * DK, nvalid, tid);
                        rawk.load_once((const bf16 *)p.k + (row0 * H + h) * DK, (long)H * DK, nvalid, tid);
                    }
                }
                if (GATED)
#pragma unroll
                    for (int j = 0; j < (int)(SM::szS / 8192); ++j) // (the reverse scan leaves -dS')
                        zs = dot8(*reinterpret_cast<const uint4 *>(blk + SM::bS + 8192 * j + 16 * tid), *reinterpret_cast<const uint4 *>(blk + SM::bDS + 8192 * j + 16 * tid), zs);
                const int kc_v = VT::kc0(lane), ks_f = frag_ks_lo(lane);
                auto rdv = [&](const unsigned char *t, int n0, int s) __attribute__((always_inline)) { return lds16(t + VT::kc(kc_v, n0, s)); };
                auto rdf = [&](const unsigned char *t, int b) __attribute__((always_inline)) { return lds_tr16(t + b * 1024 + ks_f, t + b * 1024 + (ks_f ^ 64)); };
                struct Frags { bf16x8 s, a[RB], d, u[DKW ? RB : 1]; };
                auto read = [&](Frags &f, int s) __attribute__((always_inline)) {
                    f.s = rdf(blk + SM::bS, s * (DK / 32) + kb);
                    if (DKW) {
#pragma unroll
                        for (int r = 0; r < RB; ++r) f.a[r] = rdv(blk + SM::bDV, 32 * (r ^ ti), s);
                        f.d = rdf(blk + SM::bDS, s * (DK / 32) + kb);
#pragma unroll
                        for (int r = 0; r < RB; ++r) f.u[r] = rdf(blk + SM::bUt, 2 * s + (r ^ ti));
                    } else {
#pragma unroll
                        for (int r = 0; r < RB; ++r) f.a[r] = rdv(blk + SM::bDO, 32 * (r ^ ti), s);
                        f.d = rdv(blk + SM::bDV, 32 * ti, s);
                        f.u[0] = rdf(blk + SM::bUt, 2 * s + tj);
                    }
                };
                auto products = [&](const Frags &f) __attribute__((always_inline)) {
#pragma unroll
                    for (int r = 0; r < RB; ++r) {
                        mfma32(x[r], f.s, f.a[r]);
                        if (DKW) mfma32(y[r], f.d, f.u[r]);
                    }
                    if (!DKW) { mfma32(dp, f.u[0], f.a[0]); mfma32(ah, f.u[0], f.d); }
                };
                Frags f[2];
                read(f[0], 0);
#pragma unroll
                for (int s = 0; s < KSB; ++s) {
                    if (s + 1 < KSB) read(f[(s + 1) & 1], s + 1);
                    __builtin_amdgcn_sched_barrier(0);
                    products(f[s & 1]);
                    __builtin_amdgcn_sched_barrier(0);
                }
            };
#pragma unroll
            for (int vb = 0; vb < NB; ++vb) block(vb);

            // ---- what the blocks leave
            if (masked) lds_barrier(); // dP and Ah take the bytes of V of the masked rows
            fresh();
            float zk = 0.f, z0 = 0.f; // gated: shares of <K, Ut dS~'^T> and of <Q, dO S^T> + <K, Ut dS~'^T - dV S^T>
            { // v_i . dv_i: the lanes that hold a row are adjacent
                const float s = lane_sum<VT::PPR>(cv);
                if (vp() == 0) sCv[vr()] = s;
            }
            if (masked && !DKW) {
                const float s = pm + __shfl_xor(pm, 32);
                if (lane < 32) sPm[(w4 >> 1) * C + 32 * (w4 & 1) + li] = s;
            }
            if constexpr (DKW) {
                float gm[RB];
#pragma unroll
                for (int r = 0; r < RB; ++r) {
                    gm[r] = GATED ? gamma(32 * (r ^ ti) + li) : 1.f;
                    float pr = 0.f;
#pragma unroll
                    for (int g = 0; g < 4; ++g) {
                        const f32x4 k = row4k(sK, r ^ ti, g);
#pragma unroll
                        for (int e = 0; e < 4; ++e) {
                            const float dvs = x[r][4 * g + e], uds = y[r][4 * g + e];
                            pr -= dvs * k[e];
                            if (GATED) zk -= uds * k[e];
                            y[r][4 * g + e] = -__fmaf_rn(gm[r], dvs, uds); // Ut dS'^T - dV S^T
                            if (GATED) z0 += y[r][4 * g + e] * k[e];
                        }
                    }
                    pr *= gm[r];
                    pr += __shfl_xor(pr, 32);
                    if (lane < 32) sPr[kb * C + 32 * (r ^ ti) + li] = pr;
                }
            } else {
                f32x16 l = zero16(); // k_i . k_j
                {
                    const int kc_k = KT::kc0(lane);
                    bf16x8 a[2], c[2];
                    a[0] = lds16(sK + KT::kc(kc_k, 32 * tj, 0)); c[0] = lds16(sK + KT::kc(kc_k, 32 * ti, 0));
#pragma unroll
                    for (int s = 0; s < DK / 16; ++s) {
                        if (s + 1 < DK / 16) { a[(s + 1) & 1] = lds16(sK + KT::kc(kc_k, 32 * tj, s + 1)); c[(s + 1) & 1] = lds16(sK + KT::kc(kc_k, 32 * ti, s + 1)); }
                        mfma32(l, a[s & 1], c[s & 1]);
                    }
                }
                const float gi = GATED ? gamma(32 * ti + li) : 1.f;
                if (GATED) { // the rows of dO and dV count gamma_i times
                    dp *= gi; ah *= gi;
#pragma unroll
                    for (int r = 0; r < RB; ++r) {
                        x[r] *= gamma(32 * (r ^ ti) + li);
#pragma unroll
                        for (int g = 0; g < 4; ++g) {
                            const f32x4 q = row4k(sQ, r ^ ti, g);
#pragma unroll
                            for (int e = 0; e < 4; ++e) z0 += x[r][4 * g + e] * q[e];
                        }
                    }
                }
                const int below = ti == tj ? li - 4 * hh : 64; // token i - token j of element 0 (tile (0, 1) is not used)
                float pl = 0.f;
                if (ti >= tj) {
#pragma unroll
                    for (int e = 0; e < 16; ++e) {
                        const int lower = below - 8 * (e >> 2) - (e & 3);
                        ah[e] = lower > 0 ? -ah[e] : 0.f;
                        dp[e] = lower >= 0 ? dp[e] : 0.f;
                        pl += ah[e] * l[e];
                    }
#pragma unroll
                    for (int g = 0; g < 2; ++g) {
                        const int at = (ti + tj) * (int)SM::szPT + PT::at(li, 2 * g + hh);
                        *reinterpret_cast<uint4 *>(sP + at) = row8(dp, g);
                        *reinterpret_cast<uint4 *>(sA + at) = row8(ah, g);
                    }
                    pl += __shfl_xor(pl, 32);
                    if (lane < 32) sPl[tj * C + 32 * ti + li] = pl;
                }
            }
            lds_barrier(); fresh();
            if (SM::NBUF == 1) { if (np.ok) fetch_blk(np, 0, 0); }
            else if (NB > 1 && np.ok) fetch_blk(np, 1, 1);
            const int kc_p = PT::kc0(lane), ks_k = KT::ks_lo(lane, 32 * kb), ks_p = PT::ks_lo(lane, 0);
            auto rdk = [&](const unsigned char *t, int s) __attribute__((always_inline)) { // columns 32 kb .., rows 16 s ..
                const int lo = ks_k + 16 * s * KT::RB;
                return lds_tr16(t + lo, t + KT::ks_hi(lo));
            };
            // ---- products with dP and Ah (block (i, j) of a lower triangle is tile i + j).  dQ += dP K;  dK += dP^T Q + Ah K + Ah^T K
            auto rdp = [&](const unsigned char *t, int tile, int s) __attribute__((always_inline)) { return lds16(t + tile * (int)SM::szPT + PT::kc(kc_p, 0, s)); };
            auto rdpt = [&](const unsigned char *t, int tile, int s) __attribute__((always_inline)) {
                const int lo = ks_p + tile * (int)SM::szPT + 16 * s * PT::RB;
                return lds_tr16(t + lo, t + PT::ks_hi(lo));
            };
#pragma unroll
            for (int s = 0; s < 4; ++s) { // tokens 16 s ..
                const int tb = s >> 1;
                const bf16x8 k = rdk(sK, s), q = rdk(DKW ? sQ : sK, s);
#pragma unroll
                for (int r = 0; r < RB; ++r) {
                    const int rb = r ^ ti; // token block of the result
                    if (rb >= tb) mfma32(DKW ? y[r] : x[r], k, rdp(DKW ? sA : sP, rb + tb, s & 1));
                    if (DKW && rb <= tb) {
                        mfma32(y[r], k, rdpt(sA, rb + tb, s & 1));
                        mfma32(y[r], q, rdpt(sP, rb + tb, s & 1));
                    }
                }
            }
            if (GATED && !DKW) { // q_i . dq_i, for the gate gradient
#pragma unroll
                for (int r = 0; r < RB; ++r) {
                    float cq = 0.f;
#pragma unroll
                    for (int g = 0; g < 4; ++g) {
                        const f32x4 q = row4k(sQ, r ^ ti, g);
#pragma unroll
                        for (int e = 0; e < 4; ++e) cq += x[r][4 * g + e] * q[e];
                    }
                    cq += __shfl_xor(cq, 32);
                    if (lane < 32) sCq[kb * C + 32 * (r ^ ti) + li] = cq;
                }
            }
            if (GATED) { // this wave's shares of <dS_C, S_C> and <dS_0, S_0>, summed in a fixed order after the barrier
                float zc = zk - zs, zb = z0 - zk - zs;
#pragma unroll
                for (int d = 32; d >= 1; d >>= 1) { zc += __shfl_xor(zc, d); zb += __shfl_xor(zb, d); }
                if (lane == 0) { sZ[wave] = zc; sZ[NWC + wave] = zb; }
            }
            if (!DKW && w4 == 0 && lane < nvalid) { // dbeta
                float db = sCv[lane] + sPl[lane];
                const float bt = sBeta[lane];
                if (lane >= 32) db += sPl[C + lane];
#pragma unroll
                for (int c = 0; c < NKW; ++c) db += sPr[c * C + lane];
                db = PRO ? db * (1.f - bt) : db / bt; // (prologue: through the sigmoid)
                if ((masked >> lane) & 1) {
                    db = sPm[lane] + sPm[C + lane];
                }
                p.dbeta[(row0 + lane) * H + h] = db;
            }
            lds_barrier(); fresh();
            // dQ and dK as C x d_k matrices in the bytes of Q and K, then whole rows to memory
            {
                unsigned char *to = DKW ? sK : sQ;
#pragma unroll
                for (int r = 0; r < RB; ++r)
#pragma unroll
                    for (int g = 0; g < 2; ++g)
                        *reinterpret_cast<uint4 *>(to + (32 * (r ^ ti) + li) * KT::RB + (((4 * kb + 2 * g + hh) ^ KT::swz(li)) << 4)) = row8(DKW ? y[r] : x[r], g);
            }
            if (GATED && !DKW && w4 == 0) {
                // Gate gradient.  o_t is linear in q_t and in the state, so the sensitivity to a rescaling of the state at token j
                // can be read off the other gradients: with c_i = q_i . dq_i - v_i . dv_i,
                //     dg_j = <dS_C, S_C> + sum_{i >= j} c_i = <dS_0, S_0> - sum_{i < j} c_i    (S_0, S_C: state before and after the chunk).
                // In bf16 the c_i are small differences of rounded terms and their noise adds up along the sum, so the two sums are
                // weighted by how short they are: half the error at the middle of the chunk, less towards both ends.
                float c = -sCv[lane];
#pragma unroll
                for (int b = 0; b < NKW; ++b) c += sCq[b * C + lane];
                float pre = c; // inclusive prefix sum
#pragma unroll
                for (int d = 1; d < 64; d <<= 1) {
                    const float up = __shfl_up(pre, d);
                    if (lane >= d) pre += up;
                }
                const float all = __shfl(pre, C - 1);
                auto zsum = [&](const float *z) __attribute__((always_inline)) { return ((z[0] + z[1]) + (z[2] + z[3])) + ((z[4] + z[5]) + (z[6] + z[7])); };
                const float wt = (float)lane / (float)nvalid;
                const float from_start = zsum(sZ + NWC) - (pre - c), from_end = zsum(sZ) + (all - (pre - c));
                if (lane < nvalid) p.dg[(row0 + lane) * H + h] = from_start + wt * (from_end - from_start);
            }
            lds_barrier(); fresh();
            {
                const int stride = H * DK * 2;
                const __amdgpu_buffer_rsrc_t oq = make_rsrc((bf16 *)p.dq + (row0 * H + h) * DK, nvalid * stride), ok = make_rsrc((bf16 *)p.dk + (row0 * H + h) * DK, nvalid * stride);
#pragma unroll
                for (int m = 0; m < 2; ++m)
#pragma unroll
                    for (int i = 0; i < C * KT::PPR / NTC; ++i) {
                        const int row = i * (NTC / KT::PPR) + tid / KT::PPR, piece = tid % KT::PPR;
                        u32x4 o = *reinterpret_cast<const u32x4 *>((m ? sK : sQ) + KT::at(row, piece));
                        if constexpr (PRO) o = map_gradient<KT::PPR>((m ? rawk : rawq).v[i], o);
                        __builtin_amdgcn_raw_buffer_store_b128(o, m ? ok : oq, row * stride + 16 * piece, 0, kAuxOnce);
                        if (PRO) __builtin_amdgcn_sched_barrier(0);
                    }
            }
            it = nx;
            cur = np;
            if (NB == 1) par ^= 1;
            lds_barrier(); fresh();
        }
    };
    if (wave < 4) run(std::false_type{});
    else run(std::true_type{});
}

} // namespace dn
