// One-level forward and inverse 2-D DWT kernels for gfx950.
//
// One launch computes one level: each workgroup reads its window of the level
// input once from HBM (coalesced vector loads straight into registers, the
// lifting halo included), runs every lifting step of the level in registers
// (non-separable: S_U | T_P per lifting pair, Sec. 3; separable:
// S_U^V | S_U^H | T_P^V | T_P^H, Sec. 2), scales, and writes the centre of
// the window: the four bands (forward) or the interleaved pixels (inverse).
#pragma once

#include "dwt2_device.hpp"

namespace dwt2 {

// Parameters of one forward level. The input is w x h pixels (even), the
// outputs are nqx x nqy = (w/2) x (h/2) quads per band.
struct FwdParams {
    const void *in;
    int64_t in_pitch;
    void *ll;
    int64_t ll_pitch;
    void *hl, *lh, *hh;
    int64_t band_pitch;
    int32_t w, h, nqx, nqy;
    int32_t tiles_x, tiles_y;
    int32_t vec_in, vec_ll, vec_band;   // 1: every row starts at a 32-bit word
};

struct InvParams {
    const void *ll;
    int64_t ll_pitch;
    const void *hl, *lh, *hh;
    int64_t band_pitch;
    void *out;
    int64_t out_pitch;
    int32_t w, h, nqx, nqy;
    int32_t tiles_x, tiles_y;
    uint8_t vec_ll, vec_band, vec_out;   // 1: every row starts at a 32-bit word
    uint8_t stream_out;                  // 1: vector output stores are non-temporal
};

// Whether a row of the level may start at the upper half of a word, which the
// kernels with ODD set take (RowIn, store_cols): kernels of their own, since
// in one with the word path their registers cost it wavefronts (4096^2 FP16
// forward: 16.5 us alone, 18.4 with both).
__host__ __device__ inline bool odd_rows(const FwdParams &p) { return !(p.vec_in && p.vec_ll && p.vec_band); }
__host__ __device__ inline bool odd_rows(const InvParams &p) { return !(p.vec_ll && p.vec_band && p.vec_out); }

// Geometry of a tile configuration. The horizontal halo is one lane's worth
// of quads on each side (>= the number of lifting pairs), which keeps every
// lane's loads and stores aligned to its vector width; the vertical halo is
// one quad row per lifting pair.
template <int WV, int QPL, int ROWS, int WAVES>
struct TileGeom {
    static constexpr int NP = Wavelet<WV>::NPAIRS;
    static constexpr int HX = QPL;
    static constexpr int HY = NP;
    static constexpr int OX = 64 * QPL - 2 * HX;
    static constexpr int OY = WAVES * ROWS - 2 * HY;
    static_assert(HX >= NP, "horizontal halo must cover the lifting support");
    static_assert(OY > 0, "tile too short for the lifting halo");
};

// The hardware hands consecutive workgroup ids to the 8 XCDs in turn. Remap
// the ids so that the workgroups of one XCD are numbered contiguously; with
// contiguous tile runs per workgroup, each XCD then works on one contiguous
// region of the image and the halo rows shared by neighbouring tiles stay in
// that XCD's L2.
__device__ __forceinline__ int xcd_contiguous_tile(int b, int n) {
    const int per = n >> 3, rem = n & 7;
    const int xcd = b & 7, idx = b >> 3;
    return xcd * per + (xcd < rem ? xcd : rem) + idx;
}

// Tiles are numbered row-major; with the XCD-contiguous block numbering each
// XCD sweeps one horizontal band of the level, so the rows it has in flight
// are few and whole (DRAM page locality), and horizontally adjacent tiles,
// which share partial cache lines at their edges, meet in the same L2.
__device__ __forceinline__ int block_tile() {
    return xcd_contiguous_tile(blockIdx.x, gridDim.x);
}

// ---- forward: load / store of one tile ----------------------------------------
// Column access of one lane at the level edge. A lane reads E consecutive
// elements starting at column x0; outside [0, n) each element stands for its
// symmetric-extension mirror. The mirrored columns of E consecutive positions
// lie within E consecutive indices, so two aligned E-element vector loads
// (at `base` and base + E) cover them and a per-lane select rebuilds the
// lane's values. Lanes inside the level read their E elements with the first
// load alone (the second is dropped by the buffer hardware). Every lane
// issues the same loads, so no load sits in a divergent or lane-dependent
// branch: the loads of all rows stay in flight together.
template <int E>
struct EdgeCols {
    uint32_t off_a, off_b;   // byte offsets of the two loads (kNoAccess: none)
    int sel[E];              // element k comes from index sel[k] of the 2E loaded
    bool plain;              // the lane reads its own E columns unchanged

    // m[k]: the column element k stands for (in [0, n)); plain: m[k] = x0 + k.
    template <typename T>
    __device__ __forceinline__ static EdgeCols from(const int (&m)[E], int x0, bool plain) {
        EdgeCols c;
        int lo = m[0];
#pragma unroll
        for (int k = 1; k < E; ++k) lo = min(lo, m[k]);
        c.plain = plain;
        const int base = plain ? x0 : (lo & ~(E - 1));
        c.off_a = (uint32_t)base * (uint32_t)sizeof(T);
        c.off_b = plain ? kNoAccess : (uint32_t)(base + E) * (uint32_t)sizeof(T);
#pragma unroll
        for (int k = 0; k < E; ++k) c.sel[k] = plain ? k : m[k] - base;
        return c;
    }
};

// Element i of the 2E values (a, b), as a bitwise select: exact, and kept in
// registers (a select chain over a runtime index would be lowered to an
// indexed access).
template <int E>
__device__ __forceinline__ float pick(const float (&a)[E], const float (&b)[E], int i) {
    uint32_t r = 0;
#pragma unroll
    for (int k = 0; k < E; ++k) r |= __float_as_uint(a[k]) & (0u - (uint32_t)(i == k));
#pragma unroll
    for (int k = 0; k < E; ++k) r |= __float_as_uint(b[k]) & (0u - (uint32_t)(i == E + k));
    return __uint_as_float(r);
}

// Completes the loads of `n` rows for the lanes of an edge wavefront: the
// second vector of each row, then the per-lane select. `v[r]` holds the
// first vector on entry and the lane's elements on exit.
template <typename T, int E, bool ODD, int N>
__device__ __forceinline__ void fix_cols(const RowIn<T, E, ODD> (&rows)[N], const EdgeCols<E> &c,
                                         float (&v)[N][E]) {
    float b[N][E];
#pragma unroll
    for (int r = 0; r < N; ++r) rows[r].load(c.off_b, b[r]);
#pragma unroll
    for (int r = 0; r < N; ++r) {
        float a[E];
#pragma unroll
        for (int k = 0; k < E; ++k) a[k] = v[r][k];
#pragma unroll
        for (int k = 0; k < E; ++k) v[r][k] = pick<E>(a, b[r], c.sel[k]);
    }
}

// The lane's quads start at quad column qx0 and quad row qy0 of the level;
// positions outside the level are read through the symmetric extension.
// ODD: rows may start at the upper half of a word (2-byte elements). The values
// are scaled by kFwdHeadroom<TIN>.
template <int QPL, int ROWS, typename TIN, bool ODD>
__device__ __forceinline__ void fwd_load_at(Quads<ROWS, QPL> &q, const FwdParams &prm, int qx0,
                                            int qy0) {
    constexpr float down = kFwdHeadroom<TIN>;
    const TIN *in = static_cast<const TIN *>(prm.in);
    const int px0 = 2 * qx0;
    int m[2 * QPL];
#pragma unroll
    for (int k = 0; k < 2 * QPL; ++k) m[k] = mirror(px0 + k, prm.w);
    const EdgeCols<2 * QPL> cols = EdgeCols<2 * QPL>::template from<TIN>(
        m, px0, px0 >= 0 && px0 + 2 * QPL <= prm.w);
    // all rows' first vectors, then (edge wavefronts only) the completion
    RowIn<TIN, 2 * QPL, ODD> rows[2 * ROWS];
    float v[2 * ROWS][2 * QPL];
    if (2 * qy0 >= 0 && 2 * (qy0 + ROWS) <= prm.h) {
        // all rows inside the level (wavefront-uniform): step the row pointer
        // instead of mirroring and multiplying per row, so that the loads
        // issue sooner
        const TIN *p = in + (int64_t)(2 * qy0) * prm.in_pitch;
#pragma unroll
        for (int r = 0; r < 2 * ROWS; ++r) {
            rows[r].at(p, prm.w);
            rows[r].load(cols.off_a, v[r]);
            p += prm.in_pitch;
        }
    } else {
#pragma unroll
        for (int r = 0; r < 2 * ROWS; ++r) {
            rows[r].at(in + (int64_t)mirror(2 * qy0 + r, prm.h) * prm.in_pitch, prm.w);
            rows[r].load(cols.off_a, v[r]);
        }
    }
    if (!wave_all(cols.plain)) fix_cols(rows, cols, v);
#pragma unroll
    for (int r = 0; r < ROWS; ++r) {
#pragma unroll
        for (int i = 0; i < QPL; ++i) {
            q.a[r][i] = v[2 * r][2 * i] * down; q.b[r][i] = v[2 * r][2 * i + 1] * down;
            q.c[r][i] = v[2 * r + 1][2 * i] * down; q.d[r][i] = v[2 * r + 1][2 * i + 1] * down;
        }
    }
}
template <int QPL, int ROWS, typename G, typename TIN, bool ODD>
__device__ __forceinline__ void fwd_load(Quads<ROWS, QPL> &q, const FwdParams &prm, int t,
                                         int lane, int wave) {
    const int ty = t / prm.tiles_x, tx = t - (t / prm.tiles_x) * prm.tiles_x;
    fwd_load_at<QPL, ROWS, TIN, ODD>(q, prm, tx * G::OX - G::HX + lane * QPL,
                                     ty * G::OY - G::HY + wave * ROWS);
}

template <int WV, int QPL, int ROWS, int WAVES, typename G, typename TIN, typename TLL, typename TB,
          bool ODD>
__device__ __forceinline__ void fwd_store(const Quads<ROWS, QPL> &q, const FwdParams &prm, int t,
                                          int lane, int wave) {
    using L = Wavelet<WV>;
    constexpr float up = 1.0f / kFwdHeadroom<TIN>;
    const float sLL = (float)(L::ZL * L::ZL) * up, sHL = (float)(L::ZL * L::ZH) * up;
    const float sHH = (float)(L::ZH * L::ZH) * up;
    if (lane == 0 || lane == 63) return;   // halo lanes
    const int ty = t / prm.tiles_x, tx = t - (t / prm.tiles_x) * prm.tiles_x;
    const int qx0 = tx * G::OX - G::HX + lane * QPL;
    const int qy0 = ty * G::OY - G::HY + wave * ROWS;
    TLL *ll = static_cast<TLL *>(prm.ll);
    TB *hl = static_cast<TB *>(prm.hl);
    TB *lh = static_cast<TB *>(prm.lh);
    TB *hh = static_cast<TB *>(prm.hh);
    const auto rows = [&](auto ragged) {
        constexpr bool RAGGED = decltype(ragged)::value;
        // element offsets of row qy0 + r, stepped
        int64_t rowb = (int64_t)qy0 * prm.band_pitch, rowl = (int64_t)qy0 * prm.ll_pitch;
#pragma unroll
        for (int r = 0; r < ROWS; ++r, rowb += prm.band_pitch, rowl += prm.ll_pitch) {
            const int wr = wave * ROWS + r;
            const int gy = qy0 + r;
            if (wr < G::HY || wr >= WAVES * ROWS - G::HY || gy >= prm.nqy) continue;
            float va[QPL], vb[QPL], vc[QPL], vd[QPL];
#pragma unroll
            for (int i = 0; i < QPL; ++i) {
                va[i] = q.a[r][i] * sLL; vb[i] = q.b[r][i] * sHL;
                vc[i] = q.c[r][i] * sHL; vd[i] = q.d[r][i] * sHH;
            }
            const bool on = qx0 < prm.nqx;
            store_cols<TLL, QPL, kStoreCached, RAGGED>(ll + rowl, prm.nqx, qx0, on, !ODD, va);
            store_cols<TB, QPL, kStoreCached, RAGGED>(hl + rowb, prm.nqx, qx0, on, !ODD, vb);
            store_cols<TB, QPL, kStoreCached, RAGGED>(lh + rowb, prm.nqx, qx0, on, !ODD, vc);
            store_cols<TB, QPL, kStoreCached, RAGGED>(hh + rowb, prm.nqx, qx0, on, !ODD, vd);
        }
    };
    if (sizeof(TB) == 4 || (prm.nqx & (QPL - 1)) == 0) rows(std::false_type{});
    else rows(std::true_type{});
}

// One tile of a forward level: load, lift, store. All waves of the
// workgroup call it with the same tile (it contains workgroup barriers).
template <int WV, int SCH, int QPL, int ROWS, int WAVES, typename TIN, typename TLL, typename TB,
          bool ODD>
__device__ __forceinline__ void fwd_tile(const FwdParams &prm, int t, Mailbox<QPL, WAVES> &box,
                                         int lane, int wave) {
    using G = TileGeom<WV, QPL, ROWS, WAVES>;
    Quads<ROWS, QPL> q;
    fwd_load<QPL, ROWS, G, TIN, ODD>(q, prm, t, lane, wave);
    if constexpr (SCH == NONSEP_LDS || SCH == SEP_LDS) {
        __shared__ HBox<ROWS, WAVES> hb;
        LdsExchange<ROWS, QPL, WAVES> x{&box, &hb, wave, lane, 0};
        lift_forward<WV, SCH>(q, x);
    } else {
        Exchange<ROWS, QPL, WAVES> x{&box, wave, lane, 0};
        lift_forward<WV, SCH>(q, x);
    }
    fwd_store<WV, QPL, ROWS, WAVES, G, TIN, TLL, TB, ODD>(q, prm, t, lane, wave);
}

// One tile per workgroup.
template <int WV, int SCH, int QPL, int ROWS, int WAVES, typename TIN, typename TLL, typename TB,
          bool ODD>
__global__ __launch_bounds__(64 * WAVES) void fwd_level_kernel(FwdParams prm) {
    __shared__ Mailbox<QPL, WAVES> box;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);   // uniform per wavefront
    fwd_tile<WV, SCH, QPL, ROWS, WAVES, TIN, TLL, TB, ODD>(prm, block_tile(), box, lane, wave);
}

// ---- inverse ---------------------------------------------------------------------
// Outside the level, each polyphase component is extended through the
// symmetric extension of the pixel grid it lives on: quad (i, j) component b
// stands for pixel (2i+1, 2j), and so on.
// WITH_LL false: the detail bands only (q.a is left as it is). ODD: rows may
// start at the upper half of a word (2-byte elements).
template <int QPL, int ROWS, typename TLL, typename TB, bool ODD, bool WITH_LL = true>
__device__ __forceinline__ void inv_load_at(Quads<ROWS, QPL> &q, const InvParams &prm, int qx0,
                                            int qy0) {
    const TLL *ll = static_cast<const TLL *>(prm.ll);
    const TB *hl = static_cast<const TB *>(prm.hl);
    const TB *lh = static_cast<const TB *>(prm.lh);
    const TB *hh = static_cast<const TB *>(prm.hh);
    // quad (i, j)'s even phase stands for pixel 2i, its odd phase for 2i+1
    int xe[QPL], xo[QPL];
#pragma unroll
    for (int i = 0; i < QPL; ++i) {
        xe[i] = mirror(2 * (qx0 + i), prm.w) >> 1;
        xo[i] = (mirror(2 * (qx0 + i) + 1, prm.w) - 1) >> 1;
    }
    const bool plain = qx0 >= 0 && qx0 + QPL <= prm.nqx;
    const EdgeCols<QPL> ce = EdgeCols<QPL>::template from<TB>(xe, qx0, plain);
    const EdgeCols<QPL> co = EdgeCols<QPL>::template from<TB>(xo, qx0, plain);
    const EdgeCols<QPL> cl = EdgeCols<QPL>::template from<TLL>(xe, qx0, plain);
    RowIn<TLL, QPL, ODD> rl[ROWS];                             // LL rows
    RowIn<TB, QPL, ODD> rh[ROWS], rv[ROWS], rd[ROWS];          // HL, LH, HH rows
    if (qy0 >= 0 && 2 * (qy0 + ROWS) <= prm.h) {
        // all rows inside the level (wavefront-uniform): both phases of quad
        // row gy are band row gy; step the row pointers
        const TLL *pl = ll + (int64_t)qy0 * prm.ll_pitch;
        const int64_t ob = (int64_t)qy0 * prm.band_pitch;
        const TB *ph = hl + ob, *pv = lh + ob, *pd = hh + ob;
#pragma unroll
        for (int r = 0; r < ROWS; ++r) {
            if constexpr (WITH_LL) rl[r].at(pl, prm.nqx);
            rh[r].at(ph, prm.nqx);
            rv[r].at(pv, prm.nqx);
            rd[r].at(pd, prm.nqx);
            if constexpr (WITH_LL) rl[r].load(cl.off_a, q.a[r]);
            rh[r].load(co.off_a, q.b[r]);
            rv[r].load(ce.off_a, q.c[r]);
            rd[r].load(co.off_a, q.d[r]);
            pl += prm.ll_pitch; ph += prm.band_pitch; pv += prm.band_pitch; pd += prm.band_pitch;
        }
    } else {
#pragma unroll
        for (int r = 0; r < ROWS; ++r) {
            const int gy = qy0 + r;
            const int64_t ye = mirror(2 * gy, prm.h) >> 1;
            const int64_t yo = (mirror(2 * gy + 1, prm.h) - 1) >> 1;
            if constexpr (WITH_LL) rl[r].at(ll + ye * prm.ll_pitch, prm.nqx);
            rh[r].at(hl + ye * prm.band_pitch, prm.nqx);
            rv[r].at(lh + yo * prm.band_pitch, prm.nqx);
            rd[r].at(hh + yo * prm.band_pitch, prm.nqx);
            if constexpr (WITH_LL) rl[r].load(cl.off_a, q.a[r]);
            rh[r].load(co.off_a, q.b[r]);
            rv[r].load(ce.off_a, q.c[r]);
            rd[r].load(co.off_a, q.d[r]);
        }
    }
    if (!wave_all(plain)) {
        if constexpr (WITH_LL) fix_cols(rl, cl, q.a);
        fix_cols(rh, co, q.b);
        fix_cols(rv, ce, q.c);
        fix_cols(rd, co, q.d);
    }
}
template <int QPL, int ROWS, typename G, typename TLL, typename TB, bool ODD>
__device__ __forceinline__ void inv_load(Quads<ROWS, QPL> &q, const InvParams &prm, int t,
                                         int lane, int wave) {
    const int ty = t / prm.tiles_x, tx = t - (t / prm.tiles_x) * prm.tiles_x;
    inv_load_at<QPL, ROWS, TLL, TB, ODD>(q, prm, tx * G::OX - G::HX + lane * QPL,
                                         ty * G::OY - G::HY + wave * ROWS);
}

// up: what the values are multiplied by on their way out.
template <int QPL, int ROWS, int WAVES, typename G, typename TOUT, bool ODD>
__device__ __forceinline__ void inv_store(const Quads<ROWS, QPL> &q, const InvParams &prm, int t,
                                          int lane, int wave, float up) {
    if (lane == 0 || lane == 63) return;   // halo lanes
    const int ty = t / prm.tiles_x, tx = t - (t / prm.tiles_x) * prm.tiles_x;
    const int qx0 = tx * G::OX - G::HX + lane * QPL;
    const int qy0 = ty * G::OY - G::HY + wave * ROWS;
    TOUT *out = static_cast<TOUT *>(prm.out);
    const int px0 = 2 * qx0;
    const bool on = px0 < prm.w;
    const auto rows = [&](auto policy, auto ragged) {
        constexpr int POLICY = decltype(policy)::value;
        constexpr bool RAGGED = decltype(ragged)::value;
        int64_t ro = (int64_t)(2 * qy0) * prm.out_pitch;   // pixel row 2 (qy0 + r), stepped
#pragma unroll
        for (int r = 0; r < ROWS; ++r, ro += 2 * prm.out_pitch) {
            const int wr = wave * ROWS + r;
            const int gy = qy0 + r;
            if (wr < G::HY || wr >= WAVES * ROWS - G::HY || gy >= prm.nqy) continue;
            float e[2 * QPL], o[2 * QPL];
#pragma unroll
            for (int i = 0; i < QPL; ++i) {
                e[2 * i] = q.a[r][i] * up; e[2 * i + 1] = q.b[r][i] * up;
                o[2 * i] = q.c[r][i] * up; o[2 * i + 1] = q.d[r][i] * up;
            }
            TOUT *r0 = out + ro;
            TOUT *r1 = r0 + prm.out_pitch;
            store_cols<TOUT, 2 * QPL, POLICY, RAGGED>(r0, prm.w, px0, on, !ODD, e);
            store_cols<TOUT, 2 * QPL, POLICY, RAGGED>(r1, prm.w, px0, on, !ODD, o);
        }
    };
    const std::integral_constant<int, kStoreStream> stream;
    const std::integral_constant<int, kStoreCached> cached;
    if (sizeof(TOUT) == 4 || (prm.w & (2 * QPL - 1)) == 0) {
        if (prm.stream_out) rows(stream, std::false_type{});
        else rows(cached, std::false_type{});
    } else {
        if (prm.stream_out) rows(stream, std::true_type{});
        else rows(cached, std::true_type{});
    }
}

template <int WV, int SCH, int QPL, int ROWS, int WAVES, typename TLL, typename TB, typename TOUT,
          bool ODD>
__device__ __forceinline__ void inv_tile(const InvParams &prm, int t, Mailbox<QPL, WAVES> &box,
                                         int lane, int wave) {
    using G = TileGeom<WV, QPL, ROWS, WAVES>;
    using L = Wavelet<WV>;
    constexpr float down = kInvHeadroom<TLL, TB, TOUT>;
    const float uLL = (float)(1.0 / (L::ZL * L::ZL)) * down;
    const float uHL = (float)(1.0 / (L::ZL * L::ZH)) * down;
    const float uHH = (float)(1.0 / (L::ZH * L::ZH)) * down;
    Quads<ROWS, QPL> q;
    inv_load<QPL, ROWS, G, TLL, TB, ODD>(q, prm, t, lane, wave);
#pragma unroll
    for (int r = 0; r < ROWS; ++r) {
#pragma unroll
        for (int i = 0; i < QPL; ++i) {
            q.a[r][i] *= uLL; q.b[r][i] *= uHL; q.c[r][i] *= uHL; q.d[r][i] *= uHH;
        }
    }
    if constexpr (SCH == NONSEP_LDS || SCH == SEP_LDS) {
        __shared__ HBox<ROWS, WAVES> hb;
        LdsExchange<ROWS, QPL, WAVES> x{&box, &hb, wave, lane, 0};
        lift_inverse<WV, SCH>(q, x);
    } else {
        Exchange<ROWS, QPL, WAVES> x{&box, wave, lane, 0};
        lift_inverse<WV, SCH>(q, x);
    }
    inv_store<QPL, ROWS, WAVES, G, TOUT, ODD>(q, prm, t, lane, wave, 1.0f / down);
}

template <int WV, int SCH, int QPL, int ROWS, int WAVES, typename TLL, typename TB, typename TOUT,
          bool ODD>
__global__ __launch_bounds__(64 * WAVES) void inv_level_kernel(InvParams prm) {
    __shared__ Mailbox<QPL, WAVES> box;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);   // uniform per wavefront
    inv_tile<WV, SCH, QPL, ROWS, WAVES, TLL, TB, TOUT, ODD>(prm, block_tile(), box, lane, wave);
}

// A tile of one image of several. ODD: the launch has images whose rows may start
// at odd halves; the others take the word path in it all the same.
template <int WV, int SCH, int QPL, int ROWS, int WAVES, typename TIN, typename TLL, typename TB,
          bool ODD>
__device__ __forceinline__ void fwd_image_tile(const FwdParams &prm, int t,
                                               Mailbox<QPL, WAVES> &box, int lane, int wave) {
    if (ODD && odd_rows(prm))   // workgroup-uniform
        fwd_tile<WV, SCH, QPL, ROWS, WAVES, TIN, TLL, TB, ODD>(prm, t, box, lane, wave);
    else
        fwd_tile<WV, SCH, QPL, ROWS, WAVES, TIN, TLL, TB, false>(prm, t, box, lane, wave);
}
template <int WV, int SCH, int QPL, int ROWS, int WAVES, typename TLL, typename TB, typename TOUT,
          bool ODD>
__device__ __forceinline__ void inv_image_tile(const InvParams &prm, int t,
                                               Mailbox<QPL, WAVES> &box, int lane, int wave) {
    if (ODD && odd_rows(prm))   // workgroup-uniform
        inv_tile<WV, SCH, QPL, ROWS, WAVES, TLL, TB, TOUT, ODD>(prm, t, box, lane, wave);
    else
        inv_tile<WV, SCH, QPL, ROWS, WAVES, TLL, TB, TOUT, false>(prm, t, box, lane, wave);
}

// ---- single levels of many images, parameters in the kernel arguments -----------
// Up to kBatchMax level jobs of one size class per launch (continuous
// batching: a different set of jobs every call, so nothing is planned ahead);
// their level parameters travel in the kernel arguments, and tile_start[i] is
// the first global tile index of job i (tile_start[n] is the total). One
// workgroup per tile.
constexpr int kBatchMax = 36;

struct FwdBatch {
    int32_t n;
    int32_t tile_start[kBatchMax + 1];
    FwdParams p[kBatchMax];
};
struct InvBatch {
    int32_t n;
    int32_t tile_start[kBatchMax + 1];
    InvParams p[kBatchMax];
};
static_assert(sizeof(FwdBatch) <= 4096 && sizeof(InvBatch) <= 4096, "kernel argument limit");

// Image owning global tile t (wave-uniform; the table is in kernel arguments).
template <typename B>
__device__ __forceinline__ int batch_image(const B &bt, int t) {
    int lo = 0, hi = bt.n - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (bt.tile_start[mid] <= t) lo = mid; else hi = mid - 1;
    }
    return lo;
}

template <int WV, int SCH, int QPL, int ROWS, int WAVES, typename TIN, typename TLL, typename TB,
          bool ODD>
__global__ __launch_bounds__(64 * WAVES) void fwd_batch_kernel(FwdBatch bt) {
    __shared__ Mailbox<QPL, WAVES> box;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int total = bt.tile_start[bt.n];
    for (int t = block_tile(); t < total; t += gridDim.x) {
        const int i = batch_image(bt, t);
        fwd_image_tile<WV, SCH, QPL, ROWS, WAVES, TIN, TLL, TB, ODD>(
            bt.p[i], t - bt.tile_start[i], box, lane, wave);
    }
}

template <int WV, int SCH, int QPL, int ROWS, int WAVES, typename TLL, typename TB, typename TOUT,
          bool ODD>
__global__ __launch_bounds__(64 * WAVES) void inv_batch_kernel(InvBatch bt) {
    __shared__ Mailbox<QPL, WAVES> box;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int total = bt.tile_start[bt.n];
    for (int t = block_tile(); t < total; t += gridDim.x) {
        const int i = batch_image(bt, t);
        inv_image_tile<WV, SCH, QPL, ROWS, WAVES, TLL, TB, TOUT, ODD>(
            bt.p[i], t - bt.tile_start[i], box, lane, wave);
    }
}

// ---- batches planned in a device table ------------------------------------------
// One launch covers every image of one level that uses one tile configuration,
// however many: the per-image level parameters and a tile -> image map sit in
// a table in device memory that the host planned once (a graph captures only
// the launches). Global tile t belongs to image img[t] and is that image's
// tile t - start[img[t]].
template <typename P>
struct TableLaunch {
    const int32_t *img;     // [total] image of each tile (index into params)
    const int32_t *start;   // [images] first global tile of each image
    const P *params;        // [images]
    int32_t total;          // tiles of the launch
};

// *p for a wavefront-uniform p into memory that the launch does not write, by
// scalar loads. The compiler loads it per lane (it cannot rule out that a store
// of the same loop changes it), and then takes addresses and resources made from
// it for different in every lane: loops around buffer accesses, each with a wait
// (32 images of sides up to 4096, one level from memory: FP16 inverse 28.8 us so,
// 19.7 with scalar loads in 5/3, 31.8 and 22.3 in 9/7; forward 26.2 and 22.0, 29.5
// and 25.1).
template <typename P>
__device__ __forceinline__ P load_uniform(const P *p) {
    typedef const __attribute__((address_space(4))) uint32_t Constant;
    static_assert(sizeof(P) % 4 == 0 && alignof(P) >= 4, "whole words");
    Constant *s = (Constant *)(uintptr_t)p;
    uint32_t w[sizeof(P) / 4];
#pragma unroll
    for (unsigned k = 0; k < sizeof(P) / 4; ++k) w[k] = s[k];
    P r;
    __builtin_memcpy(&r, w, sizeof r);
    return r;
}

// Every workgroup walks the tiles t = its id, id + gridDim.x, ... below
// `total`: one tile each when the grid has one workgroup per tile, several
// when the grid is capped at the resident workgroups (persistent).
template <int WV, int SCH, int QPL, int ROWS, int WAVES, typename TIN, typename TLL, typename TB,
          bool ODD>
__global__ __launch_bounds__(64 * WAVES) void fwd_table_kernel(TableLaunch<FwdParams> tl) {
    __shared__ Mailbox<QPL, WAVES> box;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    for (int t = block_tile(); t < tl.total; t += gridDim.x) {
        const int i = load_uniform(tl.img + t);
        const FwdParams prm = load_uniform(tl.params + i);
        fwd_image_tile<WV, SCH, QPL, ROWS, WAVES, TIN, TLL, TB, ODD>(
            prm, t - load_uniform(tl.start + i), box, lane, wave);
    }
}

template <int WV, int SCH, int QPL, int ROWS, int WAVES, typename TLL, typename TB, typename TOUT,
          bool ODD>
__global__ __launch_bounds__(64 * WAVES) void inv_table_kernel(TableLaunch<InvParams> tl) {
    __shared__ Mailbox<QPL, WAVES> box;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    for (int t = block_tile(); t < tl.total; t += gridDim.x) {
        const int i = load_uniform(tl.img + t);
        const InvParams prm = load_uniform(tl.params + i);
        inv_image_tile<WV, SCH, QPL, ROWS, WAVES, TLL, TB, TOUT, ODD>(
            prm, t - load_uniform(tl.start + i), box, lane, wave);
    }
}

}  // namespace dwt2
