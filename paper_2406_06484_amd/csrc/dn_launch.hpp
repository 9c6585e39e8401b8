// Launch sequences of the forward and backward pass for one (T, DK, DV); included only by the
// instantiation files.
#pragma once
#include <atomic>
#include <tuple>

#include "dn_host.hpp"
#include "dn_kernels.hpp"
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

template <typename T, int DK, int DV> size_t max_lds_bytes() {
    static_assert(PrepSmem<T, DK, DV>::bytes <= kLdsPerWorkgroup, "k_wy_prep LDS");
    static_assert(ScanFwdSmem<T, DK, DV, VBlock<T, DV, DK>::BV>::bytes <= kLdsPerWorkgroup, "k_scan_fwd LDS");
    static_assert(ScanBwdSmem<T, DK, DV, VBlock<T, DV, DK>::BV>::bytes <= kLdsPerWorkgroup, "k_scan_bwd LDS");
    static_assert(ScanFwdSmem<T, DK, DV, VBlock<T, DV, DK>::NARROW>::bytes <= ScanFwdSmem<T, DK, DV, VBlock<T, DV, DK>::BV>::bytes &&
                  ScanBwdSmem<T, DK, DV, VBlock<T, DV, DK>::NARROW>::bytes <= ScanBwdSmem<T, DK, DV, VBlock<T, DV, DK>::BV>::bytes, "narrow blocks");
    size_t m = PrepSmem<T, DK, DV>::bytes;
    if (ScanFwdSmem<T, DK, DV, VBlock<T, DV, DK>::BV>::bytes > m) m = ScanFwdSmem<T, DK, DV, VBlock<T, DV, DK>::BV>::bytes;
    if (ScanBwdSmem<T, DK, DV, VBlock<T, DV, DK>::BV>::bytes > m) m = ScanBwdSmem<T, DK, DV, VBlock<T, DV, DK>::BV>::bytes;
    static_assert(LocalSmem<T, DK, DV>::bytes_pro <= kLdsPerWorkgroup && LocalSmem<T, DK, DV>::bytes <= kLdsPerWorkgroup, "k_bwd_local LDS");
    if (LocalSmem<T, DK, DV>::bytes > m) m = LocalSmem<T, DK, DV>::bytes;
    if (LocalSmem<T, DK, DV>::bytes_pro > m) m = LocalSmem<T, DK, DV>::bytes_pro;
    return m;
}

// launches kernel<T, DK, DV, variant> for the variant the pointers ask for.  The scans know two variants
// (for the prologue they run the plain one on the q, k that k_wy_prep mapped), the chunk kernel and the reverse scan three.
#define DN_LAUNCH_SCAN(kernel, grid, nthreads, lds, ...)                                                    \
    do {                                                                                                    \
        if (p.g) DN_LAUNCH_NT((kernel<T, DK, DV, VAR_GATED>), grid, nthreads, lds, __VA_ARGS__);            \
        else DN_LAUNCH_NT((kernel<T, DK, DV, VAR_PLAIN>), grid, nthreads, lds, __VA_ARGS__);                \
    } while (0)
// ... with BV state columns per workgroup
#define DN_LAUNCH_SCAN_BV(kernel, grid, BV, lds, ...)                                                       \
    do {                                                                                                    \
        if (p.g) DN_LAUNCH_NT((kernel<T, DK, DV, VAR_GATED, BV>), grid, NTS, lds, __VA_ARGS__);             \
        else DN_LAUNCH_NT((kernel<T, DK, DV, VAR_PLAIN, BV>), grid, NTS, lds, __VA_ARGS__);                 \
    } while (0)
// ... of the reverse scan, whose dV depends on how beta was rounded and on which tokens are masked
#define DN_LAUNCH_SCAN_DV(kernel, grid, BV, lds, ...)                                                       \
    do {                                                                                                    \
        if (p.pro) DN_LAUNCH_NT((kernel<T, DK, DV, VAR_PROLOGUE, BV>), grid, NTS, lds, __VA_ARGS__);        \
        else DN_LAUNCH_SCAN_BV(kernel, grid, BV, lds, __VA_ARGS__);                                         \
    } while (0)
// Scans of few chains (`wide` = workgroups of the grid with the ordinary column blocks) run with blocks half as wide: the
// workgroups still fit the chip at once, and the step of each, whose length is the longest of a chain of products, is shorter.
// The tiles are formed by the same products in the same order, so the results are the same bits.
// Measured, d = 128, 16 heads, wide and narrow: forward pass of 1 x 1000 tokens 43.5 and 38.7 us, 4 x 2000 (the line, half the
// chip) 84.0 and 81.4, training step 101 and 92, 266 and 247; beyond the line two rounds (8 x 2048: 104 and 155 us).
// With d_k = 64 a forward pass that keeps no tiles has its line at a quarter of the chip.  Between the two, 4 x 2000 of 32 heads,
// wide and narrow: alone it is 72.7 and 69.5 us (gated 84.1 and 86.1), but a backward pass behind it loses what it gains (its
// output, in half lines, is written back then): gated, with recomputation, 275 and 276 us.  Segmented scans (sm.N > pb.N) keep
// the ordinary blocks: little to gain in their short steps (1 x 1024: forward pass 52.8 and 51.1 us, training step 112.2 and
// 113.0).  The line of the segments themselves (segment_count) is older than the narrow blocks and lies too low for short
// sequences: 1 x 1024 takes 51.5, 113 and 130 us (forward, training step, with recomputation), the uncut 1 x 1000 38.7, 92 and 97.
static inline bool narrow_blocks(const Problem &pb, const SeqMap &sm, unsigned wide, int share) {
    return sm.N == pb.N && (long)wide * share <= pb.num_cus;
}
// what the scans see: with the prologue, the mapped q and k in the workspace
static inline Ptrs scan_ptrs(const Ptrs &p) {
    Ptrs ps = p;
    if (p.pro) { ps.q = p.Qm; ps.k = p.Km; ps.pro = 0; }
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
    dim3 gchain(chain_grid(pb.N * pb.H, VBlock<T, DV, DK>::NV));
    if (int e = launch_prep<T, DK, DV>(pb, sm, p)) return e;
    Ptrs ps = scan_ptrs(p);
    if constexpr (DK == DV && DK <= 128) {
        // few long chains: cut the sequences into G segments, get every segment's start state from a first pass
        // (k_scan_state, k_seg_combine), then run the scan below over the segments side by side
        const int G = segment_count(pb.N, pb.L, pb.H, DK, DV, VBlock<T, DV, DK>::NV, pb.cu != nullptr);
        if (G > 1 && p.Sin) {
            sm.N = pb.N * G; sm.L = pb.L / G; sm.ncd = sm.L / C;
            const dim3 gseg(chain_grid(sm.N * pb.H, VBlock<T, DV, DK>::NV));
            const dim3 gstate(2 * gseg.x);
            DN_LAUNCH_SCAN(k_scan_state, gstate, NTS, (ScanFwdSmem<T, DK, DV, VBlock<T, DV, DK>::BV>::bytes), sm, pb.H, ps, (int)gseg.x);
            const CombineArgs ca{p.Mseg, p.Nseg, p.S0, p.Sin, p.ST, nullptr, nullptr, nullptr, nullptr, G, pb.H, 0};
            DN_LAUNCH_NT((k_seg_combine<DK, DV>), dim3(pb.N * pb.H, DV / 32, 1), NTHR, (CombineSmem<DK, DV>::bytes), ca);
            ps.S0 = p.Sin; ps.ST = nullptr;
            gchain = gseg;
        }
    }
    constexpr int WB = VBlock<T, DV, DK>::BV, NB = VBlock<T, DV, DK>::NARROW;
    if constexpr (NB < WB) {
        if (narrow_blocks(pb, sm, gchain.x, DK <= 64 && !pb.save ? 4 : 2)) {
            gchain.x *= WB / NB;
            if (pb.save) DN_LAUNCH_SCAN_BV(k_scan_fwd_save, gchain, NB, (ScanFwdSmem<T, DK, DV, NB>::bytes), sm, pb.H, ps);
            else DN_LAUNCH_SCAN_BV(k_scan_fwd, gchain, NB, (ScanFwdSmem<T, DK, DV, NB>::bytes), sm, pb.H, ps);
            return 0;
        }
    }
    if (pb.save) DN_LAUNCH_SCAN_BV(k_scan_fwd_save, gchain, WB, (ScanFwdSmem<T, DK, DV, WB>::bytes), sm, pb.H, ps);
    else DN_LAUNCH_SCAN_BV(k_scan_fwd, gchain, WB, (ScanFwdSmem<T, DK, DV, WB>::bytes), sm, pb.H, ps);
    return 0;
}

// the reverse scan of a backward pass, with the recompute scan in the same grid unless the forward pass left its tiles
// (gscan: the ordinary grid of one scan)
template <typename T, int DK, int DV> int launch_bwd_scans(const Problem &pb, const SeqMap &sm, const Ptrs &p, const Ptrs &ps, unsigned gscan) {
    constexpr int WB = VBlock<T, DV, DK>::BV, NB = VBlock<T, DV, DK>::NARROW;
    constexpr size_t lds_w = cmax(ScanFwdSmem<T, DK, DV, WB>::bytes, ScanBwdSmem<T, DK, DV, WB>::bytes);
    if constexpr (NB < WB) {
        if (narrow_blocks(pb, sm, pb.save ? gscan : 2 * gscan, 2)) {
            constexpr size_t lds_n = cmax(ScanFwdSmem<T, DK, DV, NB>::bytes, ScanBwdSmem<T, DK, DV, NB>::bytes);
            const unsigned half = gscan * (WB / NB);
            if (pb.save) DN_LAUNCH_SCAN_DV(k_scan_bwd, dim3(half), NB, (ScanBwdSmem<T, DK, DV, NB>::bytes), sm, pb.H, ps);
            else DN_LAUNCH_SCAN_DV(k_scan_pair, dim3(2 * half), NB, lds_n, sm, pb.H, ps, (int)half);
            return 0;
        }
    }
    if (pb.save) DN_LAUNCH_SCAN_DV(k_scan_bwd, dim3(gscan), WB, (ScanBwdSmem<T, DK, DV, WB>::bytes), sm, pb.H, ps);
    else DN_LAUNCH_SCAN_DV(k_scan_pair, dim3(2 * gscan), WB, lds_w, sm, pb.H, ps, (int)gscan);
    return 0;
}

template <typename T, int DK, int DV> int run_bwd(const Problem &pb, const Ptrs &p) {
    if (pb.N == 0) return 0;
    const SeqMap sm = make_map(pb);
    if (int e = launch_offsets(pb)) return e;
    const dim3 gchain(chain_grid(pb.N * pb.H, VBlock<T, DV, DK>::NV));
    Ptrs ps = scan_ptrs(p);
    constexpr size_t lds_pair = cmax(ScanFwdSmem<T, DK, DV, VBlock<T, DV, DK>::BV>::bytes, ScanBwdSmem<T, DK, DV, VBlock<T, DV, DK>::BV>::bytes);
    // few long chains: the scans run over G segments of the sequences side by side (see k_scan_state)
    int G = 1;
    if constexpr (DK == DV && DK <= 128) G = segment_count_bwd(pb.N, pb.L, pb.H, DK, DV, VBlock<T, DV, DK>::NV, pb.cu != nullptr);
    if (G > 1 && p.Sin && pb.chunks_ub) {
        if constexpr (DK == DV && DK <= 128) {
            SeqMap sg = sm;
            sg.N = pb.N * G; sg.L = pb.L / G; sg.ncd = sg.L / C;
            const dim3 gseg(chain_grid(sg.N * pb.H, VBlock<T, DV, DK>::NV));
            if (pb.save) { // the forward pass left its tiles and the segments' transition matrices
                DN_LAUNCH_SCAN(k_scan_bwd_state, gseg, NTS, (ScanBwdSmem<T, DK, DV, VBlock<T, DV, DK>::BV>::bytes), sg, pb.H, ps);
                const CombineArgs ca{p.Mseg, nullptr, nullptr, nullptr, nullptr, p.Rseg, p.dST, p.dSout, p.dS0, G, pb.H, 1};
                DN_LAUNCH_NT((k_seg_combine<DK, DV>), dim3(pb.N * pb.H, DV / 32, 1), NTHR, (CombineSmem<DK, DV>::bytes), ca);
                ps.dST = p.dSout; ps.dS0 = nullptr;
                if (int e = launch_bwd_scans<T, DK, DV>(pb, sg, p, ps, gseg.x)) return e;
            } else {
                if (int e = launch_prep<T, DK, DV>(pb, sm, p)) return e;
                DN_LAUNCH_SCAN(k_scan_state, dim3(3 * gseg.x), NTS, lds_pair, sg, pb.H, ps, (int)gseg.x);
                const CombineArgs ca{p.Mseg, p.Nseg, p.S0, p.Sin, nullptr, p.Rseg, p.dST, p.dSout, p.dS0, G, pb.H, 0};
                DN_LAUNCH_NT((k_seg_combine<DK, DV>), dim3(pb.N * pb.H, DV / 32, 2), NTHR, (CombineSmem<DK, DV>::bytes), ca);
                ps.S0 = p.Sin; ps.dST = p.dSout; ps.dS0 = nullptr;
                if (int e = launch_bwd_scans<T, DK, DV>(pb, sg, p, ps, gseg.x)) return e;
            }
        }
    } else if (pb.save) { // T, Ut and the chunk-initial states are the forward pass's: only the reverse scan is left
        if (int e = launch_bwd_scans<T, DK, DV>(pb, sm, p, ps, gchain.x)) return e;
    } else {
        if (pb.chunks_ub) if (int e = launch_prep<T, DK, DV>(pb, sm, p)) return e;
        // both scans of the backward pass as one grid: reverse scan first, recompute scan behind it
        if (int e = launch_bwd_scans<T, DK, DV>(pb, sm, p, ps, gchain.x)) return e;
    }
    if (pb.chunks_ub) {
        using SM = LocalSmem<T, DK, DV>;
        const long tiles = (long)pb.chunks_ub * pb.H, slots = (long)pb.num_cus * SM::WPC;
        const dim3 gpers((unsigned)(tiles < slots ? tiles : slots)); // persistent: as many workgroups as the chip holds
        if (p.g) DN_LAUNCH_NT((k_bwd_local<T, DK, DV, VAR_GATED>), gpers, NTC, SM::bytes, sm, pb.H, p, pb.chunks_ub);
        else if (p.pro) DN_LAUNCH_NT((k_bwd_local<T, DK, DV, VAR_PROLOGUE>), gpers, NTC, SM::bytes_pro, sm, pb.H, p, pb.chunks_ub);
        else DN_LAUNCH_NT((k_bwd_local<T, DK, DV, VAR_PLAIN>), gpers, NTC, SM::bytes, sm, pb.H, p, pb.chunks_ub);
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
