// Token-serial (recurrent-form) DeltaNet forward for gfx950: the delta-rule update of section 2.2
// applied one token at a time,
//
//     u_t = beta_t (v_t - S_{t-1}^T k_t),   S_t = S_{t-1} + k_t u_t^T,   o_t = S_t^T q_t,
//
// with the state in fp32 registers for the whole sequence.  This is the form the paper's speed
// comparison (section 3.3, the figure with sequence length on the x axis) measures the chunkwise
// form against, and the one a decoder runs for single-token steps.  There is no contraction wide
// enough for the matrix cores here: the work is 6 d_k fused multiply-adds per state column per token
// on the vector ALU.
//
// Mapping.  The d_v columns of the state are independent, so one wavefront owns 16 of them for one
// chain and never talks to another wavefront (no barrier).  Inside the wave, lane l = 16 * rb + j
// holds column j and the quarter rb of the d_k rows; the two reductions over d_k (S^T k and
// S^T q) finish with the two gfx950 lane swaps (v_permlane32_swap, v_permlane16_swap), which stay on
// the vector ALU.  A 16-column slice per wave gives chains * d_v / 16 waves: 1024 for 128 chains at
// d_v = 128, one per SIMD of the chip.
// Global latency (longer than a token takes) is hidden by staging: the wave fetches q, k, v, beta
// for a block of TB tokens with coalesced 16-byte loads, parks them in its private slice of LDS
// (two buffers), and works through the previous block meanwhile; all 16 lanes of a row quarter read
// the same k and q words from LDS (a broadcast, no bank conflict).  k and q are expanded to fp32 once,
// when the wave parks them, not by every one of the 16 column lanes that read them.
#include "dn_host.hpp"

namespace dn {

typedef __bf16 rbf16;

__device__ inline float rec_to_f32(float x) { return x; }
__device__ inline float rec_to_f32(rbf16 x) { return (float)x; }
__device__ inline void rec_store(float *p, float x) { *p = x; }
__device__ inline void rec_store(rbf16 *p, float x) { *p = (rbf16)x; }

// sum over the four lanes l, l ^ 16, l ^ 32, l ^ 48, delivered to all of them
__device__ inline float rec_sum4(float x) {
    const unsigned u = __float_as_uint(x);
    const auto a = __builtin_amdgcn_permlane32_swap(u, u, false, false);
    const unsigned v = __float_as_uint(__uint_as_float(a[0]) + __uint_as_float(a[1]));
    const auto b = __builtin_amdgcn_permlane16_swap(v, v, false, false);
    return __uint_as_float(b[0]) + __uint_as_float(b[1]);
}

// R consecutive elements of type T held as raw 16-byte words, expanded to fp32 on demand
template <typename T, int R> struct RowRegs {
    static constexpr int NW = R * (int)sizeof(T) / 16;
    static_assert(NW >= 1 && NW * 16 == R * (int)sizeof(T), "row slice must be whole 16-byte words");
    uint4 w[NW];
    __device__ inline void load(const T *src) { // LDS or global, 16-byte aligned
#pragma unroll
        for (int i = 0; i < NW; ++i) w[i] = reinterpret_cast<const uint4 *>(src)[i];
    }
    __device__ inline void unpack(float (&f)[R]) const {
#pragma unroll
        for (int i = 0; i < NW; ++i) {
            const unsigned d[4] = {w[i].x, w[i].y, w[i].z, w[i].w};
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                if (sizeof(T) == 4) f[4 * i + c] = __uint_as_float(d[c]);
                else { // two bf16 per dword: the fp32 value is the 16 bits moved to the top half
                    f[8 * i + 2 * c] = __uint_as_float(d[c] << 16);
                    f[8 * i + 2 * c + 1] = __uint_as_float(d[c] & 0xffff0000u);
                }
            }
        }
    }
};

constexpr int kRecCols = 16; // state columns per wavefront

// Tokens per staged block: 2 KB of k (and of q) per wave and buffer, at most 16 tokens.
template <typename T, int DK> struct RecStage {
    static constexpr int ROWB = DK * (int)sizeof(T);                  // bytes of one k or q row
    static constexpr int TB = 2048 / ROWB < 16 ? 2048 / ROWB : 16;
    static constexpr int ROWW = ROWB / 16;                            // 16-byte words per row
    static constexpr int NKW = TB * ROWW / 64;                        // k (or q) words per lane and block
    static constexpr int VROWW = kRecCols * (int)sizeof(T) / 16;      // 16-byte words of one token's v slice
    static_assert(TB >= 1 && TB * ROWW % 64 == 0 && TB * VROWW <= 64, "staging layout");
    static constexpr int ROWF = DK * 4;                               // k and q rows are parked as fp32
    static constexpr int oK = 0, oQ = TB * ROWF, oV = 2 * TB * ROWF, oB = oV + TB * kRecCols * (int)sizeof(T);
    static constexpr int oG = (oB + TB * (int)sizeof(T) + 3) & ~3;      // gated: alpha_t = exp(g_t), fp32
    static constexpr int bytes = (oG + TB * 4 + 15) & ~15;              // one buffer of one wave
};

template <typename T, int DK, bool GATED>
__global__ __launch_bounds__(256) void k_recurrent_fwd(RecArgs a) {
    using ST = RecStage<T, DK>;
    constexpr int R = DK / 4, TB = ST::TB; // rows per lane; tokens per block
    extern __shared__ __align__(16) unsigned char smem[];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int j = lane & 15, rb = lane >> 4;
    const int chain = blockIdx.x, n = chain / a.H, h = chain - n * a.H;
    const int col0 = (blockIdx.y * 4 + wave) * kRecCols, col = col0 + j;
    if (col0 >= a.DV) return; // whole wave past the last column slice (no barriers below)
    int t0, len;
    if (a.cu) { // bounded to the tensors' rows, whatever the array holds: a malformed one no host copy was there to reject stays in bounds
        t0 = min(max(a.cu[n], 0), a.L);
        len = min(max(a.cu[n + 1], t0), a.L) - t0;
    }
    else { t0 = n * a.L; len = a.L; }
    const int H = a.H, DV = a.DV;
    unsigned char *buf0 = smem + wave * 2 * ST::bytes, *buf1 = buf0 + ST::bytes;

    float S[R];
    if (a.S0) {
        const float *src = a.S0 + ((long)chain * DK + rb * R) * DV + col;
#pragma unroll
        for (int r = 0; r < R; ++r) S[r] = src[(long)r * DV];
    } else {
#pragma unroll
        for (int r = 0; r < R; ++r) S[r] = 0.f;
    }

    // one block of tokens in flight: global -> registers (fetch), registers -> LDS (park)
    uint4 gk[ST::NKW], gq[ST::NKW], gv;
    T gb;
    float ga = 1.f; // gated variant (section 6, the overview table's last row): decay alpha_t = exp(g_t) on the old state
    auto fetch = [&](int tb) __attribute__((always_inline)) { // tokens tb .. tb + TB - 1 of this sequence
#pragma unroll
        for (int i = 0; i < ST::NKW; ++i) {
            const int w = i * 64 + lane, tok = w / ST::ROWW, pos = w % ST::ROWW;
            if (tb + tok < len) {
                const long row = ((long)(t0 + tb + tok) * H + h) * DK;
                gk[i] = reinterpret_cast<const uint4 *>((const T *)a.k + row)[pos];
                gq[i] = reinterpret_cast<const uint4 *>((const T *)a.q + row)[pos];
            } else { // past the end: zeros, so that the unrolled block below multiplies finite numbers
                gk[i] = make_uint4(0, 0, 0, 0);
                gq[i] = make_uint4(0, 0, 0, 0);
            }
        }
        {
            const int tok = lane / ST::VROWW, pos = lane % ST::VROWW;
            if (tok < TB && tb + tok < len)
                gv = reinterpret_cast<const uint4 *>((const T *)a.v + ((long)(t0 + tb + tok) * H + h) * DV + col0)[pos];
            if (lane < TB && tb + lane < len) {
                gb = ((const T *)a.beta)[(long)(t0 + tb + lane) * H + h];
                if (GATED) ga = __expf(a.g[(long)(t0 + tb + lane) * H + h]);
            }
        }
    };
    auto park = [&](unsigned char *buf) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < ST::NKW; ++i) {
            constexpr int EPW = 16 / (int)sizeof(T); // elements per 16-byte word
            float fk[EPW], fq[EPW];
            RowRegs<T, EPW> wk, wq;
            wk.w[0] = gk[i]; wq.w[0] = gq[i];
            wk.unpack(fk); wq.unpack(fq);
            float *dk_ = reinterpret_cast<float *>(buf + ST::oK) + (i * 64 + lane) * EPW;
            float *dq_ = reinterpret_cast<float *>(buf + ST::oQ) + (i * 64 + lane) * EPW;
#pragma unroll
            for (int e = 0; e < EPW; e += 4) {
                *reinterpret_cast<float4 *>(dk_ + e) = make_float4(fk[e], fk[e + 1], fk[e + 2], fk[e + 3]);
                *reinterpret_cast<float4 *>(dq_ + e) = make_float4(fq[e], fq[e + 1], fq[e + 2], fq[e + 3]);
            }
        }
        if (lane < TB * ST::VROWW) reinterpret_cast<uint4 *>(buf + ST::oV)[lane] = gv;
        if (lane < TB) {
            reinterpret_cast<T *>(buf + ST::oB)[lane] = gb;
            if (GATED) reinterpret_cast<float *>(buf + ST::oG)[lane] = ga;
        }
    };

    T *op = (T *)a.o + ((long)t0 * H + h) * DV + col;
    const long sv = (long)H * DV;
    if (len > 0) { fetch(0); park(buf0); }
    if (len > TB) fetch(TB);
    for (int tb = 0; tb < len; tb += TB) {
        const unsigned char *cur = ((tb / TB) & 1) ? buf1 : buf0;
        const int nt = min(TB, len - tb);
        // Unrolled over the whole block so that the LDS reads and bf16 expansions of later tokens can
        // be scheduled under the dependent chain of earlier ones; tokens past the end of the sequence
        // leave the state alone (u = 0) and store nothing.
#pragma unroll
        for (int tt = 0; tt < TB; ++tt) {
            const bool live = tt < nt;
            RowRegs<float, R> kr, qr;
            kr.load(reinterpret_cast<const float *>(cur + ST::oK) + tt * DK + rb * R);
            qr.load(reinterpret_cast<const float *>(cur + ST::oQ) + tt * DK + rb * R);
            const float vt = rec_to_f32(reinterpret_cast<const T *>(cur + ST::oV)[tt * kRecCols + j]);
            const float bt = rec_to_f32(reinterpret_cast<const T *>(cur + ST::oB)[tt]);
            const float at = GATED ? reinterpret_cast<const float *>(cur + ST::oG)[tt] : 1.f;
            float kf[R], qf[R];
            kr.unpack(kf);
            qr.unpack(qf);
            float d0 = 0.f, d1 = 0.f, d2 = 0.f, d3 = 0.f; // S_{t-1}^T k_t, this lane's quarter of the rows
#pragma unroll
            for (int r = 0; r < R; r += 4) {
                d0 = fmaf(S[r], kf[r], d0); d1 = fmaf(S[r + 1], kf[r + 1], d1);
                d2 = fmaf(S[r + 2], kf[r + 2], d2); d3 = fmaf(S[r + 3], kf[r + 3], d3);
            }
            const float u = live ? bt * (vt - at * rec_sum4((d0 + d1) + (d2 + d3))) : 0.f;
            const float keep = live ? at : 1.f; // S_t = alpha_t S_{t-1} + k_t u_t^T
            float o0 = 0.f, o1 = 0.f, o2 = 0.f, o3 = 0.f; // S_t^T q_t, read-out from the updated state
#pragma unroll
            for (int r = 0; r < R; r += 4) {
                if (GATED) { S[r] *= keep; S[r + 1] *= keep; S[r + 2] *= keep; S[r + 3] *= keep; }
                S[r] = fmaf(kf[r], u, S[r]); o0 = fmaf(S[r], qf[r], o0);
                S[r + 1] = fmaf(kf[r + 1], u, S[r + 1]); o1 = fmaf(S[r + 1], qf[r + 1], o1);
                S[r + 2] = fmaf(kf[r + 2], u, S[r + 2]); o2 = fmaf(S[r + 2], qf[r + 2], o2);
                S[r + 3] = fmaf(kf[r + 3], u, S[r + 3]); o3 = fmaf(S[r + 3], qf[r + 3], o3);
            }
            const float out = rec_sum4((o0 + o1) + (o2 + o3));
            if (rb == 0 && live) rec_store(op, out);
            op += sv;
        }
        if (tb + TB < len) { // the block fetched during this one goes to the other buffer; request the one after it
            park(((tb / TB) & 1) ? buf0 : buf1);
            if (tb + 2 * TB < len) fetch(tb + 2 * TB);
        }
    }
    if (a.ST) {
        float *dst = a.ST + ((long)chain * DK + rb * R) * DV + col;
#pragma unroll
        for (int r = 0; r < R; ++r) dst[(long)r * DV] = S[r];
    }
}

// A few tokens on a kept state (generation): the state is read and written once and that is the time, so the lanes are laid
// out for the state's rows instead of for the token loop.  Lane l = 16 * rb + 8 * cp + e holds columns 4e .. 4e + 3 of the
// wave's 32 and, of the quarter rb of the rows, those with r % 4 in {2 cp, 2 cp + 1}: every access is 16 bytes per lane and
// whole 128-byte lines, four loads for every sixteen of k_recurrent_fwd, and no work is done for tokens that are not there (its
// block of eight is unrolled).  Each of the four partial sums over a quarter of the rows, and the order in which they are
// added, is that of k_recurrent_fwd, so a call per token and one call for all of them return the same bits.
// Waves are independent (no barrier): with few chains a workgroup is one wave, so that they spread over the chip.
// Bound by HBM: 512 states of 128 x 128 (67 MB) for one token 12.3 us, 5.4 TB/s, what a copy reaches; in k_recurrent_fwd 17.6 us.
constexpr int kDecCols = 32;
// The most tokens a call may have to come here.  A token costs this kernel about 0.7 us (its sums are spread over twice as many
// lanes) and k_recurrent_fwd next to nothing up to its block of eight, so few chains decide: 16 chains of d = 128 in bf16 take
// 3.3, 4.0, 4.7, 5.4, 6.2 us for 1 to 5 tokens against 5.4, 5.5, 5.6, 5.8, 5.9; 128 chains in fp32 5.7, 6.3, 7.3 us against 6.4,
// 6.5, 6.8.  At d_k = 256 the lanes hold 128 values of the state: 2304 chains in bf16 245, 249, 254 us against 253, 253, 252, and
// in fp32 the two are level (33.0 and 32.5 us for 256 chains), so the loop keeps it.
template <typename T, int DK> constexpr int kDecTokens = sizeof(T) == 2 ? (DK > 128 ? 2 : 4) : (DK > 128 ? 0 : 2);

template <typename T> struct DecQuad; // four neighbouring elements of v or o
template <> struct DecQuad<float> { typedef float4 raw; };
template <> struct DecQuad<rbf16> { typedef uint2 raw; };
__device__ inline void dec_unpack(const float4 &w, float (&f)[4]) { f[0] = w.x; f[1] = w.y; f[2] = w.z; f[3] = w.w; }
__device__ inline void dec_unpack(const uint2 &w, float (&f)[4]) {
    f[0] = __uint_as_float(w.x << 16); f[1] = __uint_as_float(w.x & 0xffff0000u);
    f[2] = __uint_as_float(w.y << 16); f[3] = __uint_as_float(w.y & 0xffff0000u);
}
// sum over the lanes l and l ^ 8 (a rotation by 8 inside each row of 16 lanes), then over the quarters of the rows
__device__ inline float dec_sum(float x) {
    const int o = __builtin_amdgcn_update_dpp(0, (int)__float_as_uint(x), 0x128, 0xf, 0xf, false); // row_ror:8
    return rec_sum4(x + __uint_as_float((unsigned)o));
}

template <typename T, int DK, bool GATED>
__global__ __launch_bounds__(256) void k_decode_fwd(RecArgs a) {
    constexpr int R = DK / 4, NI = R / 4;                    // rows per quarter; row pairs per lane
    constexpr int ROWW = DK * (int)sizeof(T) / 16, WT = 2 * ROWW; // 16-byte words of one k (or q) row; of a token's k and q
    constexpr int EPW = 16 / (int)sizeof(T);
    constexpr int NW = (kDecTokens<T, DK> * WT + 63) / 64;           // words per lane for all tokens
    extern __shared__ __align__(16) unsigned char smem[];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int e = lane & 7, cp = (lane >> 3) & 1, rb = lane >> 4;
    const int chain = blockIdx.x, n = chain / a.H, h = chain - n * a.H;
    const int col0 = (blockIdx.y * (blockDim.x >> 6) + wave) * kDecCols, col = col0 + 4 * e;
    const int H = a.H, DV = a.DV, len = a.L;
    if (col0 >= DV) return;
    const long t0 = (long)n * len;
    float *kq = reinterpret_cast<float *>(smem) + wave * (len * 2 * DK); // this wave's: per token k and q as fp32

    uint4 w[NW];
#pragma unroll
    for (int i = 0; i < NW; ++i) {
        const int x = i * 64 + lane, tok = x / WT, y = x % WT;
        if (tok < len) w[i] = reinterpret_cast<const uint4 *>((const T *)(y < ROWW ? a.k : a.q) + ((t0 + tok) * H + h) * DK)[y % ROWW];
    }
    typename DecQuad<T>::raw vr[kDecTokens<T, DK>];
    T br[kDecTokens<T, DK>];
    float gr[kDecTokens<T, DK>];
#pragma unroll
    for (int t = 0; t < kDecTokens<T, DK>; ++t)
        if (t < len) {
            vr[t] = *reinterpret_cast<const typename DecQuad<T>::raw *>((const T *)a.v + ((t0 + t) * H + h) * DV + col);
            br[t] = ((const T *)a.beta)[(t0 + t) * H + h];
            gr[t] = GATED ? a.g[(t0 + t) * H + h] : 0.f;
        }
    float S[2 * NI][4]; // rows rb R + 4 i + 2 cp + {0, 1}
    const long base = ((long)chain * DK + rb * R + 2 * cp) * DV + col;
#pragma unroll
    for (int i = 0; i < 2 * NI; ++i) {
        const float4 x = a.S0 ? *reinterpret_cast<const float4 *>(a.S0 + base + (long)(4 * (i >> 1) + (i & 1)) * DV) : make_float4(0.f, 0.f, 0.f, 0.f);
        S[i][0] = x.x; S[i][1] = x.y; S[i][2] = x.z; S[i][3] = x.w;
    }
#pragma unroll
    for (int i = 0; i < NW; ++i) {
        const int x = i * 64 + lane;
        if (x / WT < len) {
            float f[EPW];
            RowRegs<T, EPW> r;
            r.w[0] = w[i];
            r.unpack(f);
#pragma unroll
            for (int u = 0; u < EPW; u += 4) *reinterpret_cast<float4 *>(kq + x * EPW + u) = make_float4(f[u], f[u + 1], f[u + 2], f[u + 3]);
        }
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront"); // (parked by all lanes, read by all lanes, of the same wave)
#pragma unroll
    for (int t = 0; t < kDecTokens<T, DK>; ++t) {
        if (t >= len) break;
        const float *kt = kq + t * 2 * DK + rb * R + 2 * cp, *qt = kt + DK;
        float v[4], u[4], out[4];
        dec_unpack(vr[t], v);
        const float bt = rec_to_f32(br[t]), at = GATED ? __expf(gr[t]) : 1.f;
        float d[2][4] = {};
#pragma unroll
        for (int i = 0; i < NI; ++i) {
            const float2 kk = *reinterpret_cast<const float2 *>(kt + 4 * i);
#pragma unroll
            for (int c = 0; c < 4; ++c) { d[0][c] = fmaf(S[2 * i][c], kk.x, d[0][c]); d[1][c] = fmaf(S[2 * i + 1][c], kk.y, d[1][c]); }
        }
#pragma unroll
        for (int c = 0; c < 4; ++c) u[c] = bt * (v[c] - at * dec_sum(d[0][c] + d[1][c]));
        float o[2][4] = {};
#pragma unroll
        for (int i = 0; i < NI; ++i) {
            const float2 kk = *reinterpret_cast<const float2 *>(kt + 4 * i), qq = *reinterpret_cast<const float2 *>(qt + 4 * i);
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                if (GATED) { S[2 * i][c] *= at; S[2 * i + 1][c] *= at; }
                S[2 * i][c] = fmaf(kk.x, u[c], S[2 * i][c]);
                o[0][c] = fmaf(S[2 * i][c], qq.x, o[0][c]);
                S[2 * i + 1][c] = fmaf(kk.y, u[c], S[2 * i + 1][c]);
                o[1][c] = fmaf(S[2 * i + 1][c], qq.y, o[1][c]);
            }
        }
#pragma unroll
        for (int c = 0; c < 4; ++c) out[c] = dec_sum(o[0][c] + o[1][c]);
        if (lane < 8) {
            alignas(16) T ov[4];
#pragma unroll
            for (int c = 0; c < 4; ++c) rec_store(ov + c, out[c]);
            *reinterpret_cast<typename DecQuad<T>::raw *>((T *)a.o + ((t0 + t) * H + h) * DV + col) = *reinterpret_cast<const typename DecQuad<T>::raw *>(ov);
        }
    }
    if (a.ST) {
#pragma unroll
        for (int i = 0; i < 2 * NI; ++i)
            *reinterpret_cast<float4 *>(a.ST + base + (long)(4 * (i >> 1) + (i & 1)) * DV) = make_float4(S[i][0], S[i][1], S[i][2], S[i][3]);
    }
}

template <typename T, int DK> static int launch_decode(const RecArgs &a, hipStream_t stream) {
    const int slices = a.DV / kDecCols;
    const int waves = slices * (long)a.N * a.H <= 2048 ? 1 : (slices < 4 ? slices : 4);
    const dim3 grid(a.N * a.H, (slices + waves - 1) / waves);
    const int lds = waves * a.L * 2 * DK * (int)sizeof(float); // at most 32 KB
    void *args[] = {const_cast<RecArgs *>(&a)};
    const void *fn = a.g ? reinterpret_cast<const void *>(k_decode_fwd<T, DK, true>) : reinterpret_cast<const void *>(k_decode_fwd<T, DK, false>);
    prof_begin("k_decode_fwd", stream);
    const hipError_t e = hipLaunchKernel(fn, grid, dim3(64 * waves), args, lds, stream);
    prof_end(stream);
    return (int)e;
}

template <typename T, int DK> static int launch_rec(const RecArgs &a, hipStream_t stream) {
    if constexpr (kDecTokens<T, DK> > 0)
        if (!a.cu && a.L >= 1 && a.L <= kDecTokens<T, DK> && a.DV % kDecCols == 0) return launch_decode<T, DK>(a, stream);
    const dim3 grid(a.N * a.H, (a.DV + 4 * kRecCols - 1) / (4 * kRecCols));
    constexpr int lds = 4 * 2 * RecStage<T, DK>::bytes; // four waves, two buffers each
    static_assert(lds <= 160 * 1024, "staging fits the LDS");
    // the launch's own status (an error some earlier, unrelated call left behind is neither reported nor cleared)
    void *args[] = {const_cast<RecArgs *>(&a)};
    const void *fn = a.g ? reinterpret_cast<const void *>(k_recurrent_fwd<T, DK, true>) : reinterpret_cast<const void *>(k_recurrent_fwd<T, DK, false>);
    if (const hipError_t e = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, lds)) return (int)e;
    prof_begin("k_recurrent_fwd", stream);
    const hipError_t e = hipLaunchKernel(fn, grid, dim3(256), args, lds, stream);
    prof_end(stream);
    return (int)e;
}

// dtype: 0 = fp32, 1 = bf16.  Returns 0, a hipError_t (> 0), or -1 when (dtype, d_k) is not compiled.
int run_recurrent_fwd(int dtype, int d_k, const RecArgs &a, hipStream_t stream) {
    if (a.N == 0) return 0;
    if (dtype == 0) {
        if (d_k == 32) return launch_rec<float, 32>(a, stream);
        if (d_k == 64) return launch_rec<float, 64>(a, stream);
        if (d_k == 128) return launch_rec<float, 128>(a, stream);
        if (d_k == 256) return launch_rec<float, 256>(a, stream);
    } else {
        if (d_k == 32) return launch_rec<rbf16, 32>(a, stream);
        if (d_k == 64) return launch_rec<rbf16, 64>(a, stream);
        if (d_k == 128) return launch_rec<rbf16, 128>(a, stream);
        if (d_k == 256) return launch_rec<rbf16, 256>(a, stream);
    }
    return -1;
}

} // namespace dn
