// Fused finest levels ("head"): levels j and j+1 of a multi-level transform in
// one launch, the low-low band between them kept in registers.
//
// The finest levels carry almost all the bytes. Run one launch each, level j
// writes its low-low band to HBM and level j+1 reads it straight back, and
// each launch pays its own ramp-up and drain. Here a wavefront sweeps down a
// strip of the image and runs both levels on the rows as they pass
// (dwt2_stream.hpp). Each lane holds two quads of level j, whose low-low
// values are one quad of level j+1 in the same lane, so the band between the
// levels never leaves the lane: no LDS, and no exchange but the lane shifts.
// The same per-quad arithmetic runs on the same values as in one-level
// launches (the intermediate band is FP32 in both), so results are
// bit-identical to them.
//
// What bounds it. The bytes: a strip reads its pixels and writes its bands
// once, plus the halo (6 quads of level j on each side of what it owns). Three
// things decide how close the launch comes to the copy rate:
//   - whole lines. A strip owns OWN = 48 of its 64 lanes. So pixels and the FP32
//     bands of level j are written in pieces of 768 and 384 bytes that start on
//     a line, where the rows do; the other pieces (192 bytes, or 96) start on
//     half a line or a quarter. The halo lanes this gives up cost reads that L2
//     answers; pieces of 58 lanes (all that the halo leaves) share a line at both
//     ends with the next strip's, and lines that L2 evicts half written go out
//     twice: 16384^2 FP32 forward 486 us with 58 lanes, 443 with 48 (segments
//     of 18).
//   - lockstep. The wavefronts of a workgroup are neighbouring strips; a barrier
//     per row pair keeps them together, so that what they share (halo columns,
//     lines at piece ends) meets in L2 and the rows in flight stay few and
//     long: 463 -> 443 us at the same shape.
//   - loads far ahead. The next D - 1 row pairs are in flight while one is
//     lifted.
// By windows (dwt2_head_tile.hpp), which ran everything before, a workgroup of 12
// wavefronts lifts a 128 x 48-quad window with the low-low band in LDS: 47% more
// lifting and loads than owned quads, ten barriers per window, loads, lifting
// and stores one after the other. 16384^2 forward: 474 us FP32, 285 FP16; by
// strips 405 and 229, for bytes that the 6.2 TB/s of a large copy moves in 346 and
// 173; 4096^2 FP32 forward 37.6 -> 33.3, inverse 29.1 -> 27.2 with its bands in the
// Infinity Cache.
#pragma once

#include <type_traits>

#include "dwt2_stream.hpp"
#include "dwt2_tail.hpp"

namespace dwt2 {

// Lanes that a strip owns, row pairs it holds in registers, and strips per
// workgroup.
constexpr int kHeadOwn = 48;
constexpr int kHeadDepth = 3;
constexpr int kHeadWaves = 4;

// OWN: lanes of a strip that are written, 58 at most (both levels' halo is 6
// quads of level j, 3 lanes, on each side; 5/3 needs 3 quads).
template <int WV, int OWN>
struct HeadGeom {
    static constexpr int NP = Wavelet<WV>::NPAIRS;
    static constexpr int HALO = (64 - OWN) / 2;
    static_assert(OWN % 2 == 0 && HALO >= 3, "halo lanes");
    // row pairs a sweep starts before the first owned row of level j+1, and
    // goes on after the last
    static constexpr int F0 = NP == 2 ? 3 : 1, F1 = NP;
    static constexpr int I0 = NP == 2 ? 3 : 2, I1 = NP == 2 ? 2 : 1;
};

struct FwdHead {
    FwdParams l1;             // level j: input and detail bands (its ll is unused)
    FwdParams l2;             // level j+1: detail bands and low-low output (its in is unused)
    int32_t across;           // strips per row of tasks, or windows per row of windows
    int32_t seg;              // rows of level j+1 per segment; 0: windows (dwt2_head_tile.hpp)
};

struct InvHead {
    InvParams l2;             // level j+1: low-low and detail bands (its out is unused)
    InvParams l1;             // level j: detail bands and output (its ll is unused)
    int32_t across, seg;
};

// Whether pixel or level j band rows may start at the upper half of a word (level
// j+1 is accessed one element at a time).
__host__ __device__ inline bool odd_rows(const FwdHead &h) { return !(h.l1.vec_in && h.l1.vec_band); }
__host__ __device__ inline bool odd_rows(const InvHead &h) { return !(h.l1.vec_band && h.l1.vec_out); }

// A wavefront-uniform value that the compiler takes for another than v. The row
// loops end at the last row that is loaded; knowing that, it drops the test of
// each first load of a group and schedules the loop anew, in 130 registers
// instead of 112 (FP32 9/7 inverse: three wavefronts to a SIMD) and 114 instead of
// 106 (forward: 4096^2 34.2 us, not 33.1).
__device__ __forceinline__ int opaque(int v) {
    asm("" : "+s"(v));
    return v;
}

// One strip's segment, forward: rows o..o+seg of level j+1, the window's first
// lane at column wx. EX, EY: the window reaches the left or right (upper or
// lower) edge of the image. MODE: how rows are addressed.
//
// Iteration t takes level j rows 2t+NP-2 and 2t+NP-1 in, finishes rows 2(t-1)
// and 2(t-1)+1, which are row t-1 of level j+1, and so finishes that level's
// row t-1-NP.
template <int WV, int SCH, int OWN, typename TIN, typename TLL, typename TB, bool STREAM, bool EX,
          bool EY, int MODE>
__device__ __forceinline__ void fwd_head_strip(const FwdHead &hd, const int wx, const int o) {
    using G = HeadGeom<WV, OWN>;
    using L = Wavelet<WV>;
    constexpr int NP = G::NP, D = kHeadDepth;
    // 4-byte pixels stay in the registers of their load until their row is
    // lifted (122 registers, not 94, if both rows are scaled first); 2-byte
    // ones are decoded into others at once, and their registers can take the
    // next load a row pair earlier
    constexpr bool KEEP = sizeof(TIN) == 4;
    constexpr int AHEAD = KEEP ? D - 1 : D;
    constexpr int POLICY = STREAM ? kStoreStream : kStoreCached;
    constexpr float down = kFwdHeadroom<TIN>, up = 1.0f / down;
    const float sLL = (float)(L::ZL * L::ZL) * up, sHL = (float)(L::ZL * L::ZH) * up;
    const float sHH = (float)(L::ZH * L::ZH) * up;
    const float sL1 = (float)(L::ZL * L::ZL);             // between the levels
    const FwdParams &p1 = hd.l1, &p2 = hd.l2;
    const int lane = threadIdx.x & 63;
    const int X = wx + lane;                              // the lane's level j+1 column
    const int e = min(o + hd.seg, p2.nqy);
    const int t0 = o - G::F0, t1 = e + G::F1, tl = opaque(t1);
    const ColMarks m{X == 0, X == p2.nqx - 1};
    const bool own = lane >= G::HALO && lane < G::HALO + OWN && X < p2.nqx;
    const uint32_t offi = 4u * (uint32_t)min(max(X, 0), p2.nqx - 1) * (uint32_t)sizeof(TIN);
    const uint32_t off1 = own ? 2u * (uint32_t)X * (uint32_t)sizeof(TB) : kNoAccess;
    const uint32_t off2 = own ? (uint32_t)X * (uint32_t)sizeof(TB) : kNoAccess;
    const uint32_t offl = own ? (uint32_t)X * (uint32_t)sizeof(TLL) : kNoAccess;

    const int row0 = 4 * t0 + 2 * (NP - 2);               // first pixel row
    const RowsOf<TIN, MODE> in(p1.in, p1.in_pitch, p1.h, p1.w, EY ? max(row0, 0) : row0);
    const RowsOf<TB, MODE> hl1(p1.hl, p1.band_pitch, p1.nqy, p1.nqx, 2 * t0 - 2);
    const RowsOf<TB, MODE> lh1(p1.lh, p1.band_pitch, p1.nqy, p1.nqx, 2 * t0 - 2);
    const RowsOf<TB, MODE> hh1(p1.hh, p1.band_pitch, p1.nqy, p1.nqx, 2 * t0 - 2);
    const RowsOf<TB, MODE> hl2(p2.hl, p2.band_pitch, p2.nqy, p2.nqx, t0 - 1 - NP);
    const RowsOf<TB, MODE> lh2(p2.lh, p2.band_pitch, p2.nqy, p2.nqx, t0 - 1 - NP);
    const RowsOf<TB, MODE> hh2(p2.hh, p2.band_pitch, p2.nqy, p2.nqx, t0 - 1 - NP);
    const RowsOf<TLL, MODE> ll2(p2.ll, p2.ll_pitch, p2.nqy, p2.nqx, t0 - 1 - NP);
    uint32_t s_in = 0, s_b1 = 0, s_b2 = 0, s_ll = 0;      // row offsets, stepped

    FwdRows<WV, SCH, 2, EX, EY> v1{};
    FwdRows<WV, SCH, 1, EX, EY> v2{};
    Raw<TIN, 4, MODE> raw[D][4];
    const auto fetch = [&](int t, Raw<TIN, 4, MODE>(&w)[4]) {
        const uint32_t off = t <= t1 ? offi : kNoAccess;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const int row = 4 * t + 2 * (NP - 2) + k;
            in.template load<EY>(w[k], row, off, s_in);
            s_in += in.step;
        }
    };
#pragma unroll
    for (int i = 0; i < AHEAD; ++i) {
        fetch(t0 + i, raw[i]);
        pad_stores((KEEP && i + 1 == AHEAD) ? 7 : 10);
    }
    for (int tb = t0; tb <= tl; tb += D) {
#pragma unroll
        for (int i = 0; i < D; ++i) {
            const int t = tb + i;
            __builtin_amdgcn_s_barrier();                 // lockstep
            Line<2> x[2];
            const auto take = [&](int k) {
#pragma unroll
                for (int j = 0; j < 2; ++j) {
                    x[k].a[j] = raw[i][2 * k].get(2 * j) * down;
                    x[k].b[j] = raw[i][2 * k].get(2 * j + 1) * down;
                    x[k].c[j] = raw[i][2 * k + 1].get(2 * j) * down;
                    x[k].d[j] = raw[i][2 * k + 1].get(2 * j + 1) * down;
                }
            };
            if constexpr (!KEEP) {
                take(0);
                take(1);
                fetch(t + D, raw[i]);
            }
            __builtin_amdgcn_sched_barrier(0);
            const uint32_t o1 = (t - 1 >= o && t - 1 < e) ? off1 : kNoAccess;
#pragma unroll
            for (int k = 0; k < 2; ++k) {
                if constexpr (KEEP) take(k);
                v1.push(x[k], 2 * t + NP - 2 + k, p1.nqy, m);
                const float vb[2] = {x[k].b[0] * sHL, x[k].b[1] * sHL};
                const float vc[2] = {x[k].c[0] * sHL, x[k].c[1] * sHL};
                const float vd[2] = {x[k].d[0] * sHH, x[k].d[1] * sHH};
                const int y = 2 * t - 2 + k;
                hl1.template store<2, POLICY>(y, o1, s_b1, vb);
                lh1.template store<2, POLICY>(y, o1, s_b1, vc);
                hh1.template store<2, POLICY>(y, o1, s_b1, vd);
                s_b1 += hl1.step;
                if (KEEP && k == 0) {   // the previous pair's registers are free now
                    __builtin_amdgcn_sched_barrier(0);
                    fetch(t + D - 1, raw[(i + D - 1) % D]);
                    __builtin_amdgcn_sched_barrier(0);
                }
            }
            Line<1> q;
            q.a[0] = x[0].a[0] * sL1; q.b[0] = x[0].a[1] * sL1;
            q.c[0] = x[1].a[0] * sL1; q.d[0] = x[1].a[1] * sL1;
            v2.push(q, t - 1, p2.nqy, m);
            const int y = t - 1 - NP;
            const bool on = y >= o && y < e;
            const uint32_t o2 = on ? off2 : kNoAccess, ol = on ? offl : kNoAccess;
            const float wa[1] = {q.a[0] * sLL}, wb[1] = {q.b[0] * sHL};
            const float wc[1] = {q.c[0] * sHL}, wd[1] = {q.d[0] * sHH};
            hl2.template store<1, POLICY>(y, o2, s_b2, wb);
            lh2.template store<1, POLICY>(y, o2, s_b2, wc);
            hh2.template store<1, POLICY>(y, o2, s_b2, wd);
            ll2.template store<1>(y, ol, s_ll, wa);
            s_b2 += hl2.step;
            s_ll += ll2.step;
            __builtin_amdgcn_sched_barrier(0);
        }
    }
}

// One strip's segment, inverse. Iteration t takes row t of level j+1 in,
// finishes that level's row t-NP, which holds the low-low values of level j
// rows 2(t-NP) and 2(t-NP)+1, and so finishes level j rows 2(t-NP)-NP and
// 2(t-NP)-NP+1.
template <int WV, int SCH, int OWN, typename TLL, typename TB, typename TOUT, bool STREAM, bool EX,
          bool EY, int MODE>
__device__ __forceinline__ void inv_head_strip(const InvHead &hd, const int wx, const int o) {
    using G = HeadGeom<WV, OWN>;
    using L = Wavelet<WV>;
    constexpr int NP = G::NP, D = kHeadDepth;
    constexpr int POLICY = STREAM ? kStoreStream : kStoreCached;
    constexpr float down = kInvHeadroom<TLL, TB, TOUT>, up = 1.0f / down;
    const float uLL = (float)(1.0 / (L::ZL * L::ZL)) * down;
    const float uHL = (float)(1.0 / (L::ZL * L::ZH)) * down;
    const float uHH = (float)(1.0 / (L::ZH * L::ZH)) * down;
    const float uL1 = (float)(1.0 / (L::ZL * L::ZL));     // between the levels
    const InvParams &p1 = hd.l1, &p2 = hd.l2;
    const int lane = threadIdx.x & 63;
    const int X = wx + lane;
    const int e = min(o + hd.seg, p2.nqy);
    const int t0 = o - G::I0, t1 = e + G::I1, tl = opaque(t1);
    const ColMarks m{X == 0, X == p2.nqx - 1};
    const bool own = lane >= G::HALO && lane < G::HALO + OWN && X < p2.nqx;
    const uint32_t Xc = (uint32_t)min(max(X, 0), p2.nqx - 1);
    const uint32_t offl = Xc * (uint32_t)sizeof(TLL), off2 = Xc * (uint32_t)sizeof(TB);
    const uint32_t off1 = 2u * Xc * (uint32_t)sizeof(TB);
    const uint32_t offo = own ? 4u * (uint32_t)X * (uint32_t)sizeof(TOUT) : kNoAccess;

    const int r2 = t0, r1 = 2 * (t0 - NP), ro = 2 * (r1 - NP);   // first rows
    const RowsOf<TLL, MODE> ll(p2.ll, p2.ll_pitch, p2.nqy, p2.nqx, EY ? max(r2, 0) : r2);
    const RowsOf<TB, MODE> hl2(p2.hl, p2.band_pitch, p2.nqy, p2.nqx, EY ? max(r2, 0) : r2);
    const RowsOf<TB, MODE> lh2(p2.lh, p2.band_pitch, p2.nqy, p2.nqx, EY ? max(r2, 0) : r2);
    const RowsOf<TB, MODE> hh2(p2.hh, p2.band_pitch, p2.nqy, p2.nqx, EY ? max(r2, 0) : r2);
    const RowsOf<TB, MODE> hl1(p1.hl, p1.band_pitch, p1.nqy, p1.nqx, EY ? max(r1, 0) : r1);
    const RowsOf<TB, MODE> lh1(p1.lh, p1.band_pitch, p1.nqy, p1.nqx, EY ? max(r1, 0) : r1);
    const RowsOf<TB, MODE> hh1(p1.hh, p1.band_pitch, p1.nqy, p1.nqx, EY ? max(r1, 0) : r1);
    const RowsOf<TOUT, MODE> out(p1.out, p1.out_pitch, p1.h, p1.w, ro);
    uint32_t s_l = 0, s_2 = 0, s_1 = 0, s_o = 0;

    InvRows<WV, SCH, 1, EX, EY> v2{};
    InvRows<WV, SCH, 2, EX, EY> v1{};
    struct Pair {
        Raw<TLL, 1, MODE> a;
        Raw<TB, 1, MODE> b, c, d;
        Raw<TB, 2, MODE> fb[2], fc[2], fd[2];
    } raw[D];
    const auto fetch = [&](int t, Pair &w) {
        const bool on = t <= t1;
        const uint32_t ol = on ? offl : kNoAccess, o2 = on ? off2 : kNoAccess;
        const uint32_t o1 = on ? off1 : kNoAccess;
        ll.template load<EY>(w.a, t, ol, s_l);
        hl2.template load<EY>(w.b, t, o2, s_2);
        lh2.template load<EY>(w.c, t, o2, s_2);
        hh2.template load<EY>(w.d, t, o2, s_2);
        s_l += ll.step;
        s_2 += hl2.step;
#pragma unroll
        for (int k = 0; k < 2; ++k) {
            const int y = 2 * (t - NP) + k;
            hl1.template load<EY>(w.fb[k], y, o1, s_1);
            lh1.template load<EY>(w.fc[k], y, o1, s_1);
            hh1.template load<EY>(w.fd[k], y, o1, s_1);
            s_1 += hl1.step;
        }
    };
#pragma unroll
    for (int i = 0; i < D; ++i) {
        fetch(t0 + i, raw[i]);
        pad_stores(4);
    }
    for (int tb = t0; tb <= tl; tb += D) {
#pragma unroll
        for (int i = 0; i < D; ++i) {
            const int t = tb + i;
            __builtin_amdgcn_s_barrier();                 // lockstep
            Line<1> q;
            Line<2> x[2];
            q.a[0] = raw[i].a.get(0) * uLL; q.b[0] = raw[i].b.get(0) * uHL;
            q.c[0] = raw[i].c.get(0) * uHL; q.d[0] = raw[i].d.get(0) * uHH;
#pragma unroll
            for (int k = 0; k < 2; ++k)
#pragma unroll
                for (int j = 0; j < 2; ++j) {
                    x[k].b[j] = raw[i].fb[k].get(j) * uHL;
                    x[k].c[j] = raw[i].fc[k].get(j) * uHL;
                    x[k].d[j] = raw[i].fd[k].get(j) * uHH;
                }
            __builtin_amdgcn_sched_barrier(0);
            fetch(t + D, raw[i]);
            __builtin_amdgcn_sched_barrier(0);
            v2.push(q, t, p2.nqy, m);
            x[0].a[0] = q.a[0] * uL1; x[0].a[1] = q.b[0] * uL1;
            x[1].a[0] = q.c[0] * uL1; x[1].a[1] = q.d[0] * uL1;
#pragma unroll
            for (int k = 0; k < 2; ++k) {
                v1.push(x[k], 2 * (t - NP) + k, p1.nqy, m);
                const int y = 2 * (t - NP) - NP + k;
                const uint32_t oo = (y >= 2 * o && y < 2 * e) ? offo : kNoAccess;
                const float ev[4] = {x[k].a[0] * up, x[k].b[0] * up, x[k].a[1] * up, x[k].b[1] * up};
                out.template store<4, POLICY>(2 * y, oo, s_o, ev);
                s_o += out.step;
                // one pixel row's registers at a time: 114 in the FP32 9/7 kernel
                // instead of 130, which would leave three wavefronts to a SIMD
                __builtin_amdgcn_sched_barrier(0);
                const float od[4] = {x[k].c[0] * up, x[k].d[0] * up, x[k].c[1] * up, x[k].d[1] * up};
                out.template store<4, POLICY>(2 * y + 1, oo, s_o, od);
                s_o += out.step;
            }
            __builtin_amdgcn_sched_barrier(0);
        }
    }
}

// True when `rows` rows of `pitch` elements of T lie within one resource.
template <typename T>
__device__ __forceinline__ bool within_span(int64_t rows, int64_t pitch) {
    return rows * pitch * (int64_t)sizeof(T) < (int64_t)(kSpan / 2);
}

// Task `task` of a head: strip by strip along x, then segment by segment. A
// sweep ends with its own segment, cut off at the image's end or not: the
// barriers of the others then wait for one wavefront less, and as they guard
// no data, a wavefront that goes on to its next task may pass them out of step.
template <int WV, int SCH, int OWN, typename TIN, typename TLL, typename TB, bool STREAM>
__device__ __forceinline__ void fwd_head_task(const FwdHead &hd, const int task) {
    using G = HeadGeom<WV, OWN>;
    const int sg = task / hd.across, st = task - sg * hd.across;
    const int wx = st * OWN - G::HALO, o = sg * hd.seg;
    const FwdParams &p1 = hd.l1, &p2 = hd.l2;
    const int64_t rows = 4 * (int64_t)(hd.seg + 8 + 2 * kHeadDepth);
    const bool near = within_span<TIN>(rows, p1.in_pitch) && within_span<TB>(rows, p1.band_pitch) &&
                      within_span<TB>(rows, p2.band_pitch) && within_span<TLL>(rows, p2.ll_pitch);
    const bool vec = (sizeof(TIN) == 4 || p1.vec_in) && (sizeof(TB) == 4 || p1.vec_band);
    const bool ex = wx <= 0 || wx + 64 >= p2.nqx;
    const bool ey = o - G::F0 <= 0 || o + hd.seg + G::F1 + 1 >= p2.nqy;
    const auto run = [&](auto mode) {
        constexpr int MODE = decltype(mode)::value;
        if (ex && ey)
            fwd_head_strip<WV, SCH, OWN, TIN, TLL, TB, STREAM, true, true, MODE>(hd, wx, o);
        else if (ey)
            fwd_head_strip<WV, SCH, OWN, TIN, TLL, TB, STREAM, false, true, MODE>(hd, wx, o);
        else if (ex)
            fwd_head_strip<WV, SCH, OWN, TIN, TLL, TB, STREAM, true, false, MODE>(hd, wx, o);
        else
            fwd_head_strip<WV, SCH, OWN, TIN, TLL, TB, STREAM, false, false, MODE>(hd, wx, o);
    };
    if (!near) {
        fwd_head_strip<WV, SCH, OWN, TIN, TLL, TB, STREAM, true, true, ROWS_FAR>(hd, wx, o);
    } else if (vec) {
        run(std::integral_constant<int, ROWS_NEAR>{});
    } else {
        if constexpr (sizeof(TB) == 2) run(std::integral_constant<int, ROWS_ODD>{});
    }
}

template <int WV, int SCH, int OWN, typename TLL, typename TB, typename TOUT, bool STREAM>
__device__ __forceinline__ void inv_head_task(const InvHead &hd, const int task) {
    using G = HeadGeom<WV, OWN>;
    const int sg = task / hd.across, st = task - sg * hd.across;
    const int wx = st * OWN - G::HALO, o = sg * hd.seg;
    const InvParams &p1 = hd.l1, &p2 = hd.l2;
    const int64_t rows = 4 * (int64_t)(hd.seg + 8 + 2 * kHeadDepth);
    const bool near = within_span<TLL>(rows, p2.ll_pitch) && within_span<TB>(rows, p2.band_pitch) &&
                      within_span<TB>(rows, p1.band_pitch) && within_span<TOUT>(rows, p1.out_pitch);
    const bool vec = (sizeof(TB) == 4 || p1.vec_band) && (sizeof(TOUT) == 4 || p1.vec_out);
    const bool ex = wx <= 0 || wx + 64 >= p2.nqx;
    // the finer level's rows lag, so they reach the upper edge later
    const bool ey = o - G::I0 - G::NP <= 0 || o + hd.seg + G::I1 + 1 >= p2.nqy;
    const auto run = [&](auto mode) {
        constexpr int MODE = decltype(mode)::value;
        if (ex && ey)
            inv_head_strip<WV, SCH, OWN, TLL, TB, TOUT, STREAM, true, true, MODE>(hd, wx, o);
        else if (ey)
            inv_head_strip<WV, SCH, OWN, TLL, TB, TOUT, STREAM, false, true, MODE>(hd, wx, o);
        else if (ex)
            inv_head_strip<WV, SCH, OWN, TLL, TB, TOUT, STREAM, true, false, MODE>(hd, wx, o);
        else
            inv_head_strip<WV, SCH, OWN, TLL, TB, TOUT, STREAM, false, false, MODE>(hd, wx, o);
    };
    if (!near) {
        inv_head_strip<WV, SCH, OWN, TLL, TB, TOUT, STREAM, true, true, ROWS_FAR>(hd, wx, o);
    } else if (vec) {
        run(std::integral_constant<int, ROWS_NEAR>{});
    } else {
        if constexpr (sizeof(TB) == 2) run(std::integral_constant<int, ROWS_ODD>{});
    }
}

// This wavefront's place in the launch: the workgroup's number (XCD-contiguous)
// times the strips per workgroup, plus its own.
__device__ __forceinline__ int head_slot() {
    return block_tile() * kHeadWaves + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
}

// One image.
template <int WV, int SCH, typename TIN, typename TLL, typename TB, bool STREAM>
__global__ __launch_bounds__(64 * kHeadWaves) void fwd_head_kernel(FwdHead hd, int total) {
    const int t = head_slot();
    if (t < total) fwd_head_task<WV, SCH, kHeadOwn, TIN, TLL, TB, STREAM>(hd, t);
}

template <int WV, int SCH, typename TLL, typename TB, typename TOUT, bool STREAM>
__global__ __launch_bounds__(64 * kHeadWaves) void inv_head_kernel(InvHead hd, int total) {
    const int t = head_slot();
    if (t < total) inv_head_task<WV, SCH, kHeadOwn, TLL, TB, TOUT, STREAM>(hd, t);
}

// Heads of a planned batch: the tasks of every image in one launch, each
// image's parameters in the device copy of the plan. A workgroup walks its
// tasks in steps of the grid (several when the grid is capped at the resident
// workgroups); a wavefront that runs out ends, and no later step has work for
// it either.
template <int WV, int SCH, typename TIN, typename TLL, typename TB>
__global__ __launch_bounds__(64 * kHeadWaves) void fwd_head_table_kernel(TableLaunch<FwdHead> tl) {
    for (int t = head_slot(); t < tl.total; t += gridDim.x * kHeadWaves) {
        const int i = load_uniform(tl.img + t);
        const FwdHead hd = load_uniform(tl.params + i);
        fwd_head_task<WV, SCH, kHeadOwn, TIN, TLL, TB, false>(hd, t - load_uniform(tl.start + i));
    }
}

template <int WV, int SCH, typename TLL, typename TB, typename TOUT>
__global__ __launch_bounds__(64 * kHeadWaves) void inv_head_table_kernel(TableLaunch<InvHead> tl) {
    for (int t = head_slot(); t < tl.total; t += gridDim.x * kHeadWaves) {
        const int i = load_uniform(tl.img + t);
        const InvHead hd = load_uniform(tl.params + i);
        inv_head_task<WV, SCH, kHeadOwn, TLL, TB, TOUT, false>(hd, t - load_uniform(tl.start + i));
    }
}

// Heads of independent images in one launch, with their parameters in the
// kernel arguments (continuous batching: a different set every call), as the
// level batches: up to kHeadBatchMax heads of one set of storage types;
// tile_start[i] is the first task of head i (tile_start[n] the total).
constexpr int kHeadBatchMax = 18;

struct FwdHeadBatch {
    int32_t n;
    int32_t tile_start[kHeadBatchMax + 1];
    FwdHead h[kHeadBatchMax];
};
struct InvHeadBatch {
    int32_t n;
    int32_t tile_start[kHeadBatchMax + 1];
    InvHead h[kHeadBatchMax];
};
static_assert(sizeof(FwdHeadBatch) <= 4096 && sizeof(InvHeadBatch) <= 4096,
              "kernel argument limit");

template <int WV, int SCH, typename TIN, typename TLL, typename TB>
__global__ __launch_bounds__(64 * kHeadWaves) void fwd_head_batch_kernel(FwdHeadBatch bt) {
    const int t = head_slot();
    if (t >= bt.tile_start[bt.n]) return;
    const int i = batch_image(bt, t);
    fwd_head_task<WV, SCH, kHeadOwn, TIN, TLL, TB, false>(bt.h[i], t - bt.tile_start[i]);
}

template <int WV, int SCH, typename TLL, typename TB, typename TOUT>
__global__ __launch_bounds__(64 * kHeadWaves) void inv_head_batch_kernel(InvHeadBatch bt) {
    const int t = head_slot();
    if (t >= bt.tile_start[bt.n]) return;
    const int i = batch_image(bt, t);
    inv_head_task<WV, SCH, kHeadOwn, TLL, TB, TOUT, false>(bt.h[i], t - bt.tile_start[i]);
}

}  // namespace dwt2
