// The chunk-parallel backward kernel: everything of the backward pass that is local to one chunk, given the chunk-initial
// state S, the gradient dS' with respect to the state after the chunk, Ut (Eq. 8) and dV from the two scans.
//
// Inside a chunk Ut solves (I + A) Ut = diag(beta) (V - K S) with A = diag(beta) tril(K K^T, -1) (Eq. 10-11), so with dUt =
// P^T dO + K dS' the adjoint of the solve is G = (I + A)^-T dUt, and everything follows from G and Ut:
//     dV = diag(beta) G  (that is T^T dUt: the reverse scan forms it and stores it),    dA = -tril(G Ut^T, -1).
// The inverse of Eq. 10 and the gradients with respect to W and T never have to exist here.  Per chunk:
//     dP = tril(dO Ut^T)                  Ah = diag(beta) dA = -tril(dV Ut^T, -1)
//     dQ = dO S^T + dP K                  dK = Ut dS'^T - dV S^T + dP^T Q + (Ah + Ah^T) K
//     dbeta_i = G_i . (v_i - S_{i-1}^T k_i) = dV_i . (v_i - S^T k_i - sum_{j<i} (k_i . k_j) Ut_j) / beta_i
// In dbeta only dV carries a rounding of the row itself (v is exact, K S stays in the fp32 accumulators, Ut enters off the
// diagonal).  The shorter form dV_i . Ut_i / beta_i^2, the diagonal of dV Ut^T, has Ut_i's as well: 12 to 22 % further from the
// exact dbeta (rms, against 64 bits), 30 % in the gated variant, whose rows of dV are rounded again when they are scaled.
// Where beta is zero (a masked token), or so small that the quotient could leave the range of the types, the reverse scan has
// left dUt_i in the place of dV_i, and dbeta_i = G_i . e_i with G_i = dUt_i - sum_{j>i} (k_i . k_j) dV_j and e_i the bracket
// above; see masked_rows in the kernel.  (The prologue variant needs none of it: its gradient is that of the logit,
// dlogit_i = beta_i (1 - beta_i) G_i . e_i, which has no quotient.)
//
// This form holds the tiles on their way in registers; it is the one for fp32 and, in bf16, for d_k = 256 (see kDmaChunk).
// The operands with a d_v axis (S, dS', dO, dV, Ut) are walked in blocks of BVB state columns, each read from global memory
// once; K and Q stay in LDS for the chunk.  Every block waits in registers from the moment it is requested; as soon as it has
// moved to LDS the same registers request the block NS blocks on (of the workgroup's next chunk, at the end).
// Kernel time at 16 384 tokens of 8 heads of 256, between event records, with the shorter form of dbeta (no V, no products K S and
// K K^T) and now: 200 -> 213 us.  (The kernel that went through the inverse, with eleven barrier intervals a chunk where this one has six: 249.)
#pragma once
#include <type_traits>

#include "dn_kernels.hpp"

namespace dn {

template <typename T, int DK, int DV> struct LocalSmem {
    static constexpr int BVB0 = DK > 32 ? 32 : 64;
    static constexpr int BVB = DV < BVB0 ? DV : BVB0, NB = DV / BVB; // state columns per block, blocks per chunk
    static constexpr int NS = NB < 2 ? 1 : 2;                        // register sets for the blocks in flight
    static_assert(NB % NS == 0, "blocks alternate between the register sets");
    static constexpr int LK = ldn<T>(DK);
    static constexpr int LB = ldc<T>(BVB), LU = ldc<T>(C), LT = ldn<T>(C), LQO = ldc<T>(DK);
    static constexpr size_t oK = 0;
    static constexpr size_t oQ = oK + align16(sizeof(T) * C * LK);
    static constexpr size_t oBeta = oQ + align16(sizeof(T) * C * LK);
    static constexpr size_t oPr = oBeta + sizeof(float) * C;           // -dV_i . (K S)_i per 32 columns of a block
    static constexpr size_t oPl = oPr + sizeof(float) * (BVB / 32) * C; // -dV_i . sum_{j<i} (k_i . k_j) Ut_j per 32 tokens j
    static constexpr size_t oGam = oPl + sizeof(float) * 2 * C;        // gated: gamma_i
    static constexpr size_t oZ = oGam + sizeof(float) * C;             // gated: per-wave shares of <dS_C, S_C> and <dS_0, S_0>
    static constexpr size_t oCq = oZ + sizeof(float) * 2 * NWC;          // gated: q_i . dq_i per column block of d_k
    static constexpr size_t oCv = oCq + sizeof(float) * (DK / 32) * C; // v_i . dv_i
    // the current block ...
    static constexpr size_t oS = align16(oCv + sizeof(float) * C);
    static constexpr size_t oDS = oS + align16(sizeof(T) * BVB * LK);
    static constexpr size_t oDO = oDS + align16(sizeof(T) * BVB * LK);
    static constexpr size_t oDV = oDO + align16(sizeof(T) * C * LB);
    static constexpr size_t oUt = oDV + align16(sizeof(T) * C * LB);
    static constexpr size_t oL = oUt + align16(sizeof(T) * BVB * LU);
    // ... and for the chunks with masked rows tril(K K^T, -1) and those rows of the block as they arrived (dUt, V)
    static constexpr size_t oMD = oL + align16(sizeof(T) * C * LU), szM = align16(sizeof(T) * C * LB), oMV = oMD + szM;
    static constexpr size_t endB = oMV + szM;
    // ... and over its bytes, after the last one: dP and Ah + Ah^T, the staging tiles of the waves that own C x d_k tiles
    // (prologue variant: dq and dk as C x d_k matrices instead)
    static constexpr int TILES = 2 * (DK / 32), NSTG = TILES < NWC ? TILES : NWC;
    static constexpr size_t oDP = oS, oBm = oDP + align16(sizeof(T) * C * LT);
    static constexpr size_t oStage = oBm + align16(sizeof(T) * C * LT);
    static constexpr size_t endS = oStage + NSTG * sizeof(T) * Stage<T>::ELEMS;
    static constexpr size_t oDQm = oStage, oDKm = oDQm + align16(sizeof(T) * C * LQO), endP = oDKm + align16(sizeof(T) * C * LQO);
    static constexpr size_t bytes = cmax(endB, endS), bytes_pro = cmax(oL, endP);
};

struct NoTile {};

// A block of a tile that a scan left in the order of its operands (see dn_scan.hpp): COLS state columns of ROWS entries, in the
// LDS as COLS rows of ROWS like every other tile
template <typename T, int COLS, int ROWS, int NT> struct FragRegs {
    static constexpr int KS = Op<T>::KS, VEC = Op<T>::VEC, NS = ROWS / KS, N = COLS * ROWS / VEC, NIT = N / NT;
    static_assert(N % NT == 0, "whole rounds");
    uint4 v[NIT];
    __device__ inline void load_once(const T *src, int live, int t) {
        const __amdgpu_buffer_rsrc_t rs = make_rsrc(src);
        const int voff = live ? 16 * t : kBufRange;
#pragma unroll
        for (int it = 0; it < NIT; ++it) v[it] = buf_load16<kAuxOnce>(rs, voff, it * NT * 16);
    }
    template <bool SIGN = false> __device__ inline void store(T *dst, int ld, int t) const { // SIGN: with the sign of every element flipped
        constexpr unsigned S = !SIGN ? 0u : sizeof(T) == 2 ? 0x80008000u : 0x80000000u;
#pragma unroll
        for (int it = 0; it < NIT; ++it) {
            const int e = it * NT + t, l = e & 63, s = (e >> 6) % NS, col16 = (e >> 6) / NS;
            *reinterpret_cast<uint4 *>(dst + (16 * col16 + (l & 15)) * ld + KS * s + VEC * (l >> 4)) = make_uint4(v[it].x ^ S, v[it].y ^ S, v[it].z ^ S, v[it].w ^ S);
        }
    }
    __device__ inline float dot(const FragRegs &o) const { // sum of the products of the elements held
        float s = 0.f;
#pragma unroll
        for (int it = 0; it < NIT; ++it) {
            alignas(16) T a[VEC], b[VEC];
            *reinterpret_cast<uint4 *>(a) = v[it];
            *reinterpret_cast<uint4 *>(b) = o.v[it];
            float d = 0.f;
#pragma unroll
            for (int u = 0; u < VEC; ++u) d += to_f32(a[u]) * to_f32(b[u]);
            s += d;
        }
        return s;
    }
};

template <typename T, int DK, int DV, int VAR>
__device__ __forceinline__ void bwd_local_regs(SeqMap sm, int H, Ptrs p, int chunks_total) {
    using SM = LocalSmem<T, DK, DV>;
    constexpr bool GATED = VAR == VAR_GATED, PRO = VAR == VAR_PROLOGUE;
    constexpr int BVB = SM::BVB, NB = SM::NB;
    constexpr int NS = GATED || (PRO && DK > 128) ? 1 : SM::NS; // (the gated kernels, and the prologue's at d_k = 256, have no registers for a second set)
    constexpr int KT = SM::TILES, KW = (KT + NWC - 1) / NWC; // 32 x 32 tiles of a C x d_k matrix, and per wave
    // operand fragments per request batch (one where registers are short)
    constexpr int MB = GATED && sizeof(T) == 2 ? 1 : 2;
    // ... of the products that only dbeta needs, and of those that only masked rows need (few registers are live there)
    constexpr int MX = sizeof(T) == 4 ? 8 : 1, MM = sizeof(T) == 4 ? 8 : 4;
    // a C x BVB tile of dO, dV: 512 pieces of 16 bytes, or 256 (then each half of the workgroup fetches one of the two)
    constexpr bool HALF = C * BVB / El<T>::VEC < NTC;
    extern __shared__ __align__(16) unsigned char smem[];
    T *sK = reinterpret_cast<T *>(smem + SM::oK), *sQ = reinterpret_cast<T *>(smem + SM::oQ);
    T *sS = reinterpret_cast<T *>(smem + SM::oS), *sDS = reinterpret_cast<T *>(smem + SM::oDS);
    T *sDO = reinterpret_cast<T *>(smem + SM::oDO), *sDV = reinterpret_cast<T *>(smem + SM::oDV); // sDV holds -dV
    T *sUt = reinterpret_cast<T *>(smem + SM::oUt);
    T *sDP = reinterpret_cast<T *>(smem + SM::oDP), *sBm = reinterpret_cast<T *>(smem + SM::oBm);
    T *sL = reinterpret_cast<T *>(smem + SM::oL), *sMD = reinterpret_cast<T *>(smem + SM::oMD), *sMV = reinterpret_cast<T *>(smem + SM::oMV);
    T *sDQm = reinterpret_cast<T *>(smem + SM::oDQm), *sDKm = reinterpret_cast<T *>(smem + SM::oDKm);
    float *sBeta = reinterpret_cast<float *>(smem + SM::oBeta), *sPr = reinterpret_cast<float *>(smem + SM::oPr);
    float *sPl = reinterpret_cast<float *>(smem + SM::oPl);
    float *sGam = reinterpret_cast<float *>(smem + SM::oGam);
    float *sZ = reinterpret_cast<float *>(smem + SM::oZ), *sCq = reinterpret_cast<float *>(smem + SM::oCq), *sCv = reinterpret_cast<float *>(smem + SM::oCv);
    // The thread index as the helpers see it, re-read through an empty asm in every barrier interval: the per-lane offsets
    // derived from it are then formed where they are used instead of being carried through the whole tile loop.
    int tq = threadIdx.x;
    auto fresh = [&]() __attribute__((always_inline)) { tq = threadIdx.x; asm volatile("" : "+v"(tq)); };
    int wave = threadIdx.x >> 6;
    const bool first_half = __builtin_amdgcn_readfirstlane((int)(threadIdx.x < 256)) != 0;
    // tile number sI of this wave in a C x d_k matrix: row block ka, column block kb (with at most four such tiles they go to
    // waves 4..7: the first four waves own the C x C tiles; at d_k = 256 a wave owns both row blocks of one column block)
    constexpr int TSHIFT = KT <= 4 ? 4 : 0;
    auto kt = [&](int sI) __attribute__((always_inline)) { return TSHIFT ? ((wave + TSHIFT) & (NWC - 1)) + sI * NWC : wave + sI * NWC; };
    auto ka = [&](int sI) __attribute__((always_inline)) { return kt(sI) / (DK / 32); };
    auto kb = [&](int sI) __attribute__((always_inline)) { return kt(sI) % (DK / 32); };

    typedef TileRegs<T, C, BVB, HALF ? 256 : NTC> TokTile; // a block of dO, dV or V
    static_assert(TokTile::NIT == 1 || sizeof(T) == 4 || !HALF, "one row per thread");
    struct Blk {
        FragRegs<T, BVB, DK, NTC> s, ds;
        TokTile a;                                            // dO (HALF: first half dO, second half dV)
        std::conditional_t<HALF, NoTile, TokTile> b;          // dV
        FragRegs<T, BVB, C, HALF ? 256 : NTC> ut;             // (HALF: both halves hold a copy, the first one stores it)
        TokTile v;                                            // V, for v_i . dv_i (HALF: in the second half, beside dV)
        float gr[TokTile::NIT];                               // gated: gamma of this thread's rows
    } r[NS];
    struct Head {
        TileRegs<T, C, DK, NTC> k, q;
        T beta; // kept in storage format: converting here would wait for the whole prefetch
        float gm;
    } rh;
    std::conditional_t<PRO, TileRegs<T, C, DK, NTC>, NoTile> rawq, rawk;
    // (`live` = 0 masks every row of a request: the instruction is issued, no memory is touched; no branch stands around a
    // request, so the compiler knows how many are in flight and waits for exactly the one it needs)
    auto fetch_blk = [&](Blk &x, const TilePos &tp, int vb, int live) __attribute__((always_inline)) {
        const int v0 = vb * BVB, tt = HALF ? (tq & 255) : tq;
        const long row = (tp.row0 * H + tp.h) * DV + v0, tv = tp.tile * DV + v0;
        x.s.load_once((const T *)p.Sc + tv * DK, live, tq);
        x.ds.load_once((const T *)p.dSc + tv * DK, live, tq);
        if constexpr (HALF) x.a.load_once((first_half ? (const T *)p.d_o : (const T *)p.dv) + row, (long)H * DV, tp.nvalid * live, tt);
        else {
            x.a.load_once((const T *)p.d_o + row, (long)H * DV, tp.nvalid * live, tq);
            x.b.load_once((const T *)p.dv + row, (long)H * DV, tp.nvalid * live, tq);
        }
        x.ut.load_once((const T *)p.Ut + tv * C, live, tt);
        x.v.load_once((const T *)p.v + row, (long)H * DV, HALF && first_half ? 0 : tp.nvalid * live, tt);
        if constexpr (GATED) x.a.load_row_factors(x.gr, p.gam + tp.tile * 2 * C, tt);
    };
    auto fetch_head = [&](const TilePos &tp, int live) __attribute__((always_inline)) {
        // (prologue variant: the q and k that k_wy_prep mapped and left in the workspace, in the layout of q and k)
        rh.k.load_once((const T *)(PRO ? p.Km : p.k) + (tp.row0 * H + tp.h) * DK, (long)H * DK, tp.nvalid * live, tq);
        rh.q.load_once((const T *)(PRO ? p.Qm : p.q) + (tp.row0 * H + tp.h) * DK, (long)H * DK, tp.nvalid * live, tq);
        rh.beta = ((const T *)p.beta)[(tp.row0 + min(tq & 63, tp.nvalid - 1)) * H + tp.h]; // (every wave: each looks for masked rows)
        if (GATED && tq < C) rh.gm = p.gam[tp.tile * 2 * C + tq];
    };
    auto pos_of = [&](const TileIter &it) __attribute__((always_inline)) { return it.valid() ? tile_pos(sm, H, it.gid(), it.head()) : TilePos{0, 0, 0, 0, false}; };

    TileIter it(chunks_total, H);
    TilePos cur = pos_of(it);
    if (cur.ok) {
        fetch_head(cur, 1);
#pragma unroll
        for (int s = 0; s < NS; ++s) fetch_blk(r[s], cur, s, 1);
    }
    while (cur.ok) { // packed layout: the first chunk past the last real one ends the walk (so would every later one)
        TileIter nx = it;
        nx.next();
        const TilePos np = pos_of(nx);
        const TilePos nf = np.ok ? np : cur; // what the freed registers request at the end (masked where there is no next chunk)
        const int nl = np.ok ? 1 : 0;
        asm volatile("" : "+v"(wave)); // opaque: the tile offsets derived from it are not hoisted out of the loop
        const int mi = (wave >> 1) & 1, ni = wave & 1; // tile of every C x C matrix, for the first four waves
        const bool cc = wave < 4, upper = (mi == 0 && ni == 1);
        T *stg = reinterpret_cast<T *>(smem + SM::oStage) + (wave % SM::NSTG) * Stage<T>::ELEMS;
        const int nvalid = cur.nvalid, h = cur.h;
        const long row0 = cur.row0;

        rh.k.store(sK, SM::LK, tq); rh.q.store(sQ, SM::LK, tq);
        float b = (tq & 63) < nvalid ? to_f32(rh.beta) : 0.f;
        if (PRO) b = (tq & 63) < nvalid ? sigmoid_f32(b) : 0.f; // beta = sigmoid(logit), section 2.2
        const unsigned long long masked = PRO ? 0ull : __ballot((tq & 63) < nvalid && fabsf(b) < kTinyBeta); // the same in every wave
        if (tq < C) {
            sBeta[tq] = b;
            if (GATED) sGam[tq] = rh.gm;
        }
        // prologue variant: the pre-activations, for the way back through the map at the end of the chunk (at d_k = 256 they are
        // requested after the last block: there are no registers to hold them longer)
        auto fetch_raw = [&]() __attribute__((always_inline)) {
            if constexpr (PRO) {
                rawq.load_once((const T *)p.q + (row0 * H + h) * DK, (long)H * DK, nvalid, tq);
                rawk.load_once((const T *)p.k + (row0 * H + h) * DK, (long)H * DK, nvalid, tq);
            }
        };
        if (DK <= 128) fetch_raw();
        if (DK <= 128) fetch_head(nf, nl);
        // gated: this thread's shares of <dS~', S_0> and <K, Ut dS~'^T>
        float zs = 0.f, zk = 0.f;
        f32x16 dpc = zero16(), ahc = zero16(), dq[KW], dk[KW];
        // (where the C x C tiles and the C x d_k tiles are on different waves, they share registers)
        f32x16 &dp = TSHIFT ? dq[0] : dpc, &ah = TSHIFT ? dk[0] : ahc;
        // The tiles of (K S)^T (BVB x C) go to the waves with less to do in a block, tile kst to token block ua, column block ub:
        // the first ones, if others own the C x d_k tiles, and otherwise those that own no C x C tile, in the registers of one.
        // (Transposed: the lane's column is a token, so the sum over the state columns is over its own registers.)
        const int kst = TSHIFT ? wave : wave - 4, ua = kst / (BVB / 32), ub = kst % (BVB / 32);
        const bool does_ks = kst >= 0 && kst < 2 * (BVB / 32);
        f32x16 ksx = zero16(), gx = zero16();
        f32x16 &ks = TSHIFT ? ksx : dpc, &g = TSHIFT ? gx : ahc;
        float pr = 0.f;
#pragma unroll
        for (int sI = 0; sI < KW; ++sI) { dq[sI] = zero16(); dk[sI] = zero16(); }

        // dbeta and dV of the masked rows, over the columns of block vb, by the waves that have just formed (K S)^T: the
        // accumulators of a lane are 16 columns of its token i, so each of
        //     e_i = v_i - S^T k_i - sum_{j<i} (k_i . k_j) Ut_j,   G_i = dUt_i - sum_{j>i} (k_i . k_j) dV_j
        // is one more product with tril(K K^T, -1) and four loads per lane, and G_i . e_i a sum over registers.  In sDV the masked rows
        // are zero so far (dV_i = beta_i G_i, and beta_i is zero but for the tiny ones, which are filled in at the end).
        // Ut_i = beta_i e_i holds for them as for any row, so nothing else of the chunk is touched.  A training step on 16 384
        // tokens of width 2048 without masked tokens, with a tenth of them masked, and padded to twice the shortest length:
        // d = 128 383, 404, 388 us (a second walk over the chunks with masked rows: 363, 1569, 965), d = 64 403, 437, 426,
        // d = 256 705, 737, 734, gated 486, 519, 501.
        auto masked_rows = [&](int vb) __attribute__((always_inline)) {
            if (vb == 0) {
                if (cc) {
                    f32x16 l = zero16();
                    if (!upper) mma<DK, false, false, T, true, MX>(l, sK + 32 * mi * SM::LK, SM::LK, sK + 32 * ni * SM::LK, SM::LK, tq);
                    acc_each(l, [&](int rr, int c, float &val) { if (32 * mi + rr <= 32 * ni + c) val = 0.f; }, tq);
                    acc_to_lds<T>(sL, SM::LU, 32 * mi, 32 * ni, l, tq);
                }
                lds_barrier(); fresh();
            }
            const int lane = tq & 63, i = 32 * ua + (lane & 31), v0 = 32 * ub + 4 * (lane >> 5); // token, first column
            const bool mine = does_ks && ((masked >> (i & 63)) & 1);
            const float bi = sBeta[i & (C - 1)];
            if (does_ks) {
                const long at = ((row0 + i) * H + h) * DV + vb * BVB + v0;
                mma<C, false, false, T, true, MM>(ks, sUt + 32 * ub * SM::LU, SM::LU, sL + 32 * ua * SM::LU, SM::LU, tq); // + (tril(K K^T, -1) Ut)^T
                g = zero16();
                mma<C, true, true, T, true, MM>(g, sDV + 32 * ub, SM::LB, sL + 32 * ua, SM::LU, tq); // -(tril(K K^T, -1)^T dV)^T
                if (mine) {
                    float gm = 1.f, gi = 1.f; // gated: the tiles are in the chunk's coordinates
                    if (GATED) { gm = sGam[i]; gi = p.gam[cur.tile * 2 * C + C + i]; }
#pragma unroll
                    for (int u = 0; u < 4; ++u) {
                        T du[4], vv[4], out[4];
                        ld4(du, sMD + i * SM::LB + v0 + 8 * u);
                        ld4(vv, sMV + i * SM::LB + v0 + 8 * u);
#pragma unroll
                        for (int w = 0; w < 4; ++w) {
                            const int el = 4 * u + w;
                            g[el] += to_f32(du[w]) * gm;
                            pr += g[el] * (to_f32(vv[w]) * gi - ks[el]);
                            g[el] *= bi;
                            out[w] = from_f32<T>(g[el] * gi);
                        }
                        st4v((T *)p.dv + at + 8 * u, out);
                        __builtin_amdgcn_sched_barrier(0);
                    }
                }
            }
            if (__ballot((tq & 63) < nvalid && ((masked >> (tq & 63)) & 1) && sBeta[tq & 63] != 0.f)) {
                lds_barrier(); fresh();
                if (mine)
#pragma unroll
                    for (int u = 0; u < 4; ++u) st4(sDV + i * SM::LB + v0 + 8 * u, -g[4 * u], -g[4 * u + 1], -g[4 * u + 2], -g[4 * u + 3]);
                lds_barrier(); fresh();
            }
        };
        auto block = [&](Blk &x, int vb) __attribute__((always_inline)) {
            { // v_i . dv_i over this block's columns: the lanes that hold a row are adjacent
                const int tt = HALF ? (tq & 255) : tq;
                if (masked) {
#pragma unroll
                    for (int i = 0; i < TokTile::NIT; ++i) {
                        const int row = i * TokTile::RPI + tt / TokTile::TPR;
                        if (((masked >> row) & 1) && (!HALF || !first_half)) {
                            uint4 *d;
                            if constexpr (HALF) d = x.a.v + i;
                            else d = x.b.v + i;
                            *reinterpret_cast<uint4 *>(sMD + row * SM::LB + (tt % TokTile::TPR) * El<T>::VEC) = *d;
                            *reinterpret_cast<uint4 *>(sMV + row * SM::LB + (tt % TokTile::TPR) * El<T>::VEC) = x.v.v[i];
                            *d = make_uint4(0, 0, 0, 0);
                        }
                    }
                }
#pragma unroll
                for (int i = 0; i < TokTile::NIT; ++i) {
                    float s;
                    if constexpr (HALF) s = x.a.dot_row(x.v, i);
                    else s = x.b.dot_row(x.v, i);
                    s = lane_sum<TokTile::TPR>(s);
                    if (tt % TokTile::TPR == 0 && (!HALF || !first_half)) {
                        float *to = sCv + i * TokTile::RPI + tt / TokTile::TPR;
                        *to = vb == 0 ? s : *to + s;
                    }
                }
            }
            // gated: the chunk is the plain rule on v_i / gamma_i with outputs gamma_i o~_i, so dO and dV rows come in scaled by gamma_i
            if constexpr (GATED) {
                zs -= x.ds.dot(x.s);
                x.a.scale_rows(x.gr);
                if constexpr (!HALF) x.b.scale_rows(x.gr);
            }
            x.s.store(sS, SM::LK, tq); x.ds.template store<true>(sDS, SM::LK, tq); // (the reverse scan leaves -dS')
            if constexpr (HALF) {
                if (first_half) { x.a.store(sDO, SM::LB, tq & 255); x.ut.store(sUt, SM::LU, tq & 255); }
                else x.a.store_neg(sDV, SM::LB, tq & 255);
            } else {
                x.a.store(sDO, SM::LB, tq); x.b.store_neg(sDV, SM::LB, tq);
                x.ut.store(sUt, SM::LU, tq);
            }
            // this set's registers are free again
            const bool wrap = vb + NS >= NB;
            fetch_blk(x, wrap ? nf : cur, wrap ? vb + NS - NB : vb + NS, wrap ? nl : 1);
            lds_barrier(); fresh();
            if (does_ks) { // (K S)^T, and its products with -dV
                ks = zero16();
                mma<DK, false, false, T, true, MX>(ks, sS + 32 * ub * SM::LK, SM::LK, sK + 32 * ua * SM::LK, SM::LK, tq);
                acc_each4(ks, [&](int v, int i, float a, float b, float c, float d) {
                    T x[4];
                    ld4(x, sDV + (32 * ua + i) * SM::LB + 32 * ub + v);
                    pr += (a * to_f32(x[0]) + b * to_f32(x[1])) + (c * to_f32(x[2]) + d * to_f32(x[3]));
                }, tq);
                __builtin_amdgcn_sched_barrier(0);
            }
            if (masked) masked_rows(vb);
            if (cc && !upper) // dO Ut^T, -dV Ut^T: the fragments of Ut are read once for both
                mma_shared_b<BVB, false, false, true, T, MB>(dp, ah, sDO + 32 * mi * SM::LB, SM::LB, sDV + 32 * mi * SM::LB, SM::LB, sUt + 32 * ni, SM::LU, tq);
#pragma unroll
            for (int sI = 0; sI < KW; ++sI) if (kt(sI) < KT) {
                // dO S^T, -dV S^T
                mma_shared_b<BVB, false, false, true, T, MB>(dq[sI], dk[sI], sDO + 32 * ka(sI) * SM::LB, SM::LB, sDV + 32 * ka(sI) * SM::LB, SM::LB,
                                                             sS + 32 * kb(sI), SM::LK, tq);
                if (GATED) { // Ut dS~'^T on its own, for <K, Ut dS~'^T>
                    f32x16 t = zero16();
                    mma<BVB, true, true, T, true, MB>(t, sUt + 32 * ka(sI), SM::LU, sDS + 32 * kb(sI), SM::LK, tq);
                    acc_each(t, [&](int rr, int c, float &val) { zk += val * to_f32(sK[(32 * ka(sI) + rr) * SM::LK + 32 * kb(sI) + c]); }, tq);
                    __builtin_amdgcn_sched_barrier(0);
                    dk[sI] += t;
                } else {
                    mma<BVB, true, true, T, true, MB>(dk[sI], sUt + 32 * ka(sI), SM::LU, sDS + 32 * kb(sI), SM::LK, tq);
                }
            }
            lds_barrier(); fresh(); // the block's bytes are free
        };
        if constexpr (NB == NS) {
#pragma unroll
            for (int vb = 0; vb < NB; ++vb) block(r[vb], vb);
        } else {
#pragma unroll 1
            for (int vb = 0; vb < NB; vb += NS) {
                block(r[0], vb);
                if (NS == 2) block(r[NS - 1], vb + 1);
            }
        }
        if (does_ks) {
            pr += __shfl_xor(pr, 32);
            if ((tq & 63) < 32) sPr[ub * C + 32 * ua + (tq & 31)] = pr;
        }
                    if (cc && !upper) { // -dV_i . sum_{j<i} (k_i . k_j) Ut_j
                        f32x16 l = zero16();
                        mma<DK, false, false, T, true, MX>(l, sK + 32 * mi * SM::LK, SM::LK, sK + 32 * ni * SM::LK, SM::LK, tq);
                        const int lane = tq & 63, below = 32 * (mi - ni) + 4 * (lane >> 5) - (lane & 31); // row - column of element 0
        #pragma unroll
                        for (int e = 0; e < 16; ++e) l[e] = below + 8 * (e >> 2) + (e & 3) > 0 ? l[e] * ah[e] : 0.f;
                        row_sums(sPl + ni * C + 32 * mi, l, tq);
                    }
        if (DK > 128) fetch_raw();
        if (DK > 128) fetch_head(nf, nl); // (no registers to hold it longer)

        float z0 = 0.f; // gated: this thread's share of <Q, dO S^T> + <K, Ut dS~'^T - dV S^T>
        if (GATED) {
#pragma unroll
            for (int sI = 0; sI < KW; ++sI) if (kt(sI) < KT) {
                acc_each(dq[sI], [&](int rr, int c, float &val) { z0 += val * to_f32(sQ[(32 * ka(sI) + rr) * SM::LK + 32 * kb(sI) + c]); }, tq);
                __builtin_amdgcn_sched_barrier(0);
                acc_each(dk[sI], [&](int rr, int c, float &val) { z0 += val * to_f32(sK[(32 * ka(sI) + rr) * SM::LK + 32 * kb(sI) + c]); }, tq);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
        if (cc) {
            // dP = tril(dO Ut^T); Bm = Ah + Ah^T with Ah = -tril(dV Ut^T, -1)
            if (mi == ni) {
                const int lane = tq & 63, c = lane & 31, hh = lane >> 5;
#pragma unroll
                for (int e = 0; e < 16; ++e) {
                    const int rr = 8 * (e >> 2) + 4 * hh + (e & 3), i = 32 * mi + rr, j = 32 * mi + c;
                    if (rr >= c) {
                        const T x = from_f32<T>(rr == c ? 0.f : ah[e]);
                        sBm[i * SM::LT + j] = x;
                        sBm[j * SM::LT + i] = x;
                    }
                    dp[e] = rr >= c ? dp[e] : 0.f;
                }
            } else if (mi == 1) {
                acc_to_lds<T>(sBm, SM::LT, 32, 0, ah, tq);
                acc_to_lds_t<T>(sBm, SM::LT, 32, 0, ah, tq);
            }
            acc_to_lds<T>(sDP, SM::LT, 32 * mi, 32 * ni, dp, tq); // (the upper tile: zero)
        }
        lds_barrier(); fresh();
#pragma unroll
        for (int sI = 0; sI < KW; ++sI) if (kt(sI) < KT) {
            // dQ += dP K, dK += Bm K (shared fragments of K), dK += dP^T Q (dP is lower triangular)
            mma_shared_b<C, false, false, true, T, MB>(dq[sI], dk[sI], sDP + 32 * ka(sI) * SM::LT, SM::LT, sBm + 32 * ka(sI) * SM::LT, SM::LT,
                                                       sK + 32 * kb(sI), SM::LK, tq);
            if (ka(sI) == 1) mma<32, true, true, T, true, MB>(dk[sI], sDP + 32 * SM::LT + 32, SM::LT, sQ + 32 * SM::LK + 32 * kb(sI), SM::LK, tq);
            else mma<C, true, true, T, true, MB>(dk[sI], sDP, SM::LT, sQ + 32 * kb(sI), SM::LK, tq);
            if (PRO) {
                acc_to_lds<T>(sDQm, SM::LQO, 32 * ka(sI), 32 * kb(sI), dq[sI], tq);
                acc_to_lds<T>(sDKm, SM::LQO, 32 * ka(sI), 32 * kb(sI), dk[sI], tq);
            } else {
                if (GATED) { // also q_i . dq_i over this tile's columns, for the gate gradient
                    acc_to_lds<T>(stg, Stage<T>::LD, 0, 0, dq[sI], tq);
                    stage_flush_dot<T>(stg, (T *)p.dq + (row0 * H + h) * DK, (long)H * DK, 32 * ka(sI), 32 * kb(sI), nvalid, sQ, SM::LK,
                                       sCq + kb(sI) * C);
                } else {
                    acc_store<T, true>(stg, (T *)p.dq + (row0 * H + h) * DK, (long)H * DK, 32 * ka(sI), 32 * kb(sI), nvalid, dq[sI], tq);
                }
                acc_store<T, true>(stg, (T *)p.dk + (row0 * H + h) * DK, (long)H * DK, 32 * ka(sI), 32 * kb(sI), nvalid, dk[sI], tq);
            }
        }
        if (tq < nvalid) { // (nvalid <= C) dbeta
            float db = sCv[tq] + sPl[tq];
            if (tq >= 32) db += sPl[C + tq];
#pragma unroll
            for (int c = 0; c < BVB / 32; ++c) db += sPr[c * C + tq];
            const float b = sBeta[tq];
            db = PRO ? db * (1.f - b) : ((masked >> tq) & 1) ? db : db / b; // (prologue: through the sigmoid)
            p.dbeta[(row0 + tq) * H + h] = db;
        }
        if (GATED) { // this wave's shares of <dS_C, S_C> and <dS_0, S_0>, summed in a fixed order after the barrier
            float zc = zs + zk, zb = zs - zk + z0;
#pragma unroll
            for (int d = 32; d >= 1; d >>= 1) { zc += __shfl_xor(zc, d); zb += __shfl_xor(zb, d); }
            if ((tq & 63) == 0) { sZ[wave] = zc; sZ[NWC + wave] = zb; }
        }
        lds_barrier(); fresh();
        if constexpr (PRO) { // dq, dk are assembled: gradient through the feature map, dx = SiLU'(x) (dy - y (y . dy)) / ||SiLU(x)||
            rawq.feature_map_bwd_store(sDQm, SM::LQO, (T *)p.dq + (row0 * H + h) * DK, (long)H * DK, nvalid, tq);
            rawk.feature_map_bwd_store(sDKm, SM::LQO, (T *)p.dk + (row0 * H + h) * DK, (long)H * DK, nvalid, tq);
            lds_barrier(); fresh();
        }
        if (GATED && tq < C) {
            // Gate gradient.  o_t is linear in q_t and in the state, so the sensitivity to a rescaling of the state at token j
            // can be read off the other gradients: with c_i = q_i . dq_i - v_i . dv_i,
            //     dg_j = <dS_C, S_C> + sum_{i >= j} c_i = <dS_0, S_0> - sum_{i < j} c_i    (S_0, S_C: state before and after the chunk).
            // In bf16 the c_i are small differences of rounded terms and their noise adds up along the sum, so the two sums are
            // weighted by how short they are: half the error at the middle of the chunk, less towards both ends.
            float c = -sCv[tq];
#pragma unroll
            for (int b = 0; b < DK / 32; ++b) c += sCq[b * C + tq];
            float pre = c; // inclusive prefix sum
#pragma unroll
            for (int d = 1; d < 64; d <<= 1) {
                const float up = __shfl_up(pre, d);
                if (tq >= d) pre += up;
            }
            const float all = __shfl(pre, C - 1);
            auto zsum = [&](const float *z) __attribute__((always_inline)) { return ((z[0] + z[1]) + (z[2] + z[3])) + ((z[4] + z[5]) + (z[6] + z[7])); };
            const float w = (float)tq / (float)nvalid;
            const float from_start = zsum(sZ + NWC) - (pre - c), from_end = zsum(sZ) + (all - (pre - c));
            if (tq < nvalid) p.dg[(row0 + tq) * H + h] = from_start + w * (from_end - from_start);
        }
        if (GATED) { lds_barrier(); fresh(); }
        it = nx;
        cur = np;
    }
}

} // namespace dn
