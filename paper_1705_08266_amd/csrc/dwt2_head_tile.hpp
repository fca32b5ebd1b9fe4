// Fused finest levels by windows ("tiles"), for images too small to fill the
// chip with strips.
//
// One workgroup computes level j over a window of 128 x 48 quads, two per lane
// (the one-level kernels' register tile and lifting code), keeps the scaled
// low-low values that its window produces correctly in LDS, and computes level
// j+1 from them over the co-located coarser window. Per-quad arithmetic and
// values are those of the strips (dwt2_head.hpp) and of one-level launches, so
// results are the same bits.
//
// Against the strips: a window has its halo on all four sides, and its load,
// lifting and store phases follow each other, which costs where a compute unit
// runs many. But its 12 wavefronts start all their loads at once and lift
// four rows each, where a strip walks its rows one after the other, six of
// them halo: as long as every window is resident at once, the launch is over
// sooner. 3072^2 inverse with its bands in the caches: FP32 14.6 us against
// 17.2, FP16 13.0 against 17.6; 2048^2 FP16 forward 11.4 against 12.5
// (4096^2, FP32 inverse: 39.8 against 33.2).
//
// Geometry, with a halo unit RG = 2 quads (at least the number of lifting
// pairs of either wavelet), in quads of each level:
//   forward: the coarser window is 62 x H2 quads (lanes 0..61, each one quad,
//     H2 rows over the wavefronts), of which the centre 58 x (H2 - 2 RG) is
//     owned. It reads the low-low values of 124 x 2 H2 finer quads, the part
//     of the finer 128 x NR1 window (one halo lane and RG halo rows on each
//     side) that the finer lifting computes correctly; so NR1 = 2 H2 + 2 RG.
//     The finer level writes the bands of its 116 x 2 (H2 - 2 RG) quads that
//     map to the owned coarser block.
//   inverse: the finer window is 120 x NR1 quads (lanes 0..59; lanes 60..63
//     carry nothing useful), of which the centre 116 x (NR1 - 2 RG) is written.
//     It needs the finer low-low band over its whole window, i.e. coarser
//     outputs over 60 x NR1/2 quads; the coarser window adds RG on each side:
//     64 x (NR1/2 + 2 RG) quads.
// Outside the image each level reads its input through the whole-sample
// symmetric extension (forward) or the per-phase extension of the
// coefficients (inverse), as the one-level kernels do; the mirrored
// positions of every value that reaches a written output fall inside the
// region held in LDS, and reads for other lanes are clamped into it.
#pragma once

#include "dwt2_head.hpp"

namespace dwt2 {

// 12 wavefronts of 4 quad rows. Rows that may start at odd halves have kernels of
// their own, as in the one-level launches.
constexpr int kHeadTileRows = 4, kHeadTileWaves = 12;

template <int ROWS, int WAVES>
struct WindowGeom {
    static constexpr int RG = 2;
    static constexpr int NR1 = WAVES * ROWS;              // finer window rows
    static_assert(NR1 % 2 == 0, "whole coarser rows");
    // forward
    static constexpr int FH2 = (NR1 - 2 * RG) / 2;        // coarser window rows
    static constexpr int FOX2 = 62 - 2 * RG;              // coarser owned columns
    static constexpr int FOY2 = FH2 - 2 * RG;             // coarser owned rows
    static constexpr int FROWS2 = (FH2 + WAVES - 1) / WAVES;
    static_assert(FOY2 > 0, "forward head window too short");
    // inverse
    static constexpr int IOX1 = 116;                      // finer owned columns
    static constexpr int IOY1 = NR1 - 2 * RG;             // finer owned rows
    static constexpr int IH2 = NR1 / 2 + 2 * RG;          // coarser window rows
    static constexpr int IROWS2 = (IH2 + WAVES - 1) / WAVES;
};

// Position p of an LDS axis of n values starting at p0, clamped into it.
__device__ __forceinline__ int lds_at(int p, int p0, int n) { return min(max(p - p0, 0), n - 1); }

// Wavefronts per SIMD that the register allocation must allow. Two head
// workgroups share a CU (their LDS fits twice), which takes WAVES/2 per SIMD,
// i.e. at most 80 VGPRs for 12 wavefronts; with 81 one runs on a CU, about 35%
// slower. Left free, forward heads of BF16 rows that may start at odd halves come
// out at 87 (held to the budget 80 and 8-16 bytes spilled), all others at 56-80.
template <int SCH, int WAVES, typename TIN>
constexpr int kFwdHeadWavesPerSimd = sizeof(TIN) == 2 ? (2 * WAVES + 3) / 4 : (WAVES + 3) / 4;
template <int WAVES>
constexpr int kInvHeadWavesPerSimd = (WAVES + 3) / 4;
// The planned heads (which read their parameters from memory, one more register
// or so) are all held to the two-workgroup budget.
template <int WAVES>
constexpr int kTableHeadWavesPerSimd = (2 * WAVES + 3) / 4;

// LDS of a head workgroup: the mailbox serves the finer level's exchanges, then
// the coarser level's (smaller); ll1 holds the level j low-low band as the four
// components of the level j+1 quads, [phase][row][column].
template <int WAVES, int H2>
struct TileLds {
    Mailbox<2, WAVES> box;
    float ll1[4][H2][64];
};

template <int ROWS, int WAVES>
using FwdTileLds = TileLds<WAVES, WindowGeom<ROWS, WAVES>::FH2>;
template <int ROWS, int WAVES>
using InvTileLds = TileLds<WAVES, WindowGeom<ROWS, WAVES>::IH2>;

// Levels j and j+1 of forward window t (row-major, hd.across to a row). ODD:
// rows may start at the upper half of a word (2-byte elements).
// Wavefronts below the coarser level's window return early, after passing its
// barriers.
template <int WV, int SCH, int ROWS, int WAVES, typename TIN, typename TLL, typename TB, bool ODD>
__device__ __forceinline__ void fwd_head_tile(const FwdHead &hd, const int t,
                                              FwdTileLds<ROWS, WAVES> &lds) {
    using G = WindowGeom<ROWS, WAVES>;
    using L = Wavelet<WV>;
    constexpr int RG = G::RG, H2 = G::FH2, R2 = G::FROWS2, NR1 = G::NR1;
    Mailbox<2, WAVES> &box = lds.box;
    float(&ll1)[4][H2][64] = lds.ll1;
    constexpr float up = 1.0f / kFwdHeadroom<TIN>;
    const float sLL = (float)(L::ZL * L::ZL) * up, sHL = (float)(L::ZL * L::ZH) * up;
    const float sHH = (float)(L::ZH * L::ZH) * up;
    const float sL1 = (float)(L::ZL * L::ZL);           // between the levels
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int ty = t / hd.across, tx = t - ty * hd.across;
    const int ox2 = tx * G::FOX2, oy2 = ty * G::FOY2;   // owned block of level j+1

    // ---- level j: window of 128 x NR1 quads, two per lane
    {
        const FwdParams &p1 = hd.l1;
        const int qx = 2 * (ox2 - RG - 1 + lane);       // the lane's first quad column
        const int qy0 = 2 * oy2 - 3 * RG + wave * ROWS; // its first quad row
        Quads<ROWS, 2> q;
        fwd_load_at<2, ROWS, TIN, ODD>(q, p1, qx, qy0);
        {
            Exchange<ROWS, 2, WAVES> x{&box, wave, lane, 0};
            lift_forward<WV, SCH>(q, x);
        }
        // correct low-low values (lanes 1..62, rows RG..NR1-RG-1) into LDS
        if (lane >= 1 && lane <= 62) {
#pragma unroll
            for (int r = 0; r < ROWS; ++r) {
                const int rr = wave * ROWS + r - RG;
                if (rr >= 0 && rr < 2 * H2) {
                    const int ph = 2 * (rr & 1);
                    ll1[ph][rr >> 1][lane - 1] = q.a[r][0] * sL1;
                    ll1[ph + 1][rr >> 1][lane - 1] = q.a[r][1] * sL1;
                }
            }
        }
        __syncthreads();   // the low-low band is in LDS; every level j exchange is done
        // detail bands of the quads under the owned level j+1 block, issued
        // after the barrier so that no wavefront waits there for another's
        // store addressing
        const bool own_x = lane >= RG + 1 && lane < RG + 1 + G::FOX2 && qx + 2 <= p1.nqx;
        TB *hl = static_cast<TB *>(p1.hl);
        TB *lh = static_cast<TB *>(p1.lh);
        TB *hh = static_cast<TB *>(p1.hh);
        int64_t rowo = (int64_t)qy0 * p1.band_pitch;   // band row qy0 + r, stepped
#pragma unroll
        for (int r = 0; r < ROWS; ++r, rowo += p1.band_pitch) {
            const int wr = wave * ROWS + r;
            const int gy = qy0 + r;
            if (wr < 3 * RG || wr >= 3 * RG + 2 * G::FOY2 || gy >= p1.nqy) continue;
            const float vb[2] = {q.b[r][0] * sHL, q.b[r][1] * sHL};
            const float vc[2] = {q.c[r][0] * sHL, q.c[r][1] * sHL};
            const float vd[2] = {q.d[r][0] * sHH, q.d[r][1] * sHH};
            store_cols<TB, 2, kStoreCached, false>(hl + rowo, p1.nqx, qx, own_x, !ODD, vb);
            store_cols<TB, 2, kStoreCached, false>(lh + rowo, p1.nqx, qx, own_x, !ODD, vc);
            store_cols<TB, 2, kStoreCached, false>(hh + rowo, p1.nqx, qx, own_x, !ODD, vd);
        }
    }

    // ---- level j+1: window of 62 x H2 quads, one per lane, R2 rows per wavefront
    const FwdParams &p2 = hd.l2;
    if (wave * R2 >= H2) {   // below the window: pass the lifting's barriers
        idle_through_lifting<WV>();
        return;
    }
    const int c0 = ox2 - RG, r0 = oy2 - RG;             // LDS origin, level j+1 quads
    const int X = c0 + lane;
    const int xe = mirror(2 * X, p2.w), xo = mirror(2 * X + 1, p2.w);
    const int ce = lds_at(xe >> 1, c0, 62), co = lds_at(xo >> 1, c0, 62);
    Quads<R2, 1> q;
    const int Y0 = r0 + wave * R2;
    if (Y0 >= 0 && 2 * (Y0 + R2) <= p2.h) {
        // all rows inside the level (wavefront-uniform): no row is mirrored
#pragma unroll
        for (int r = 0; r < R2; ++r) {
            const int ry = lds_at(Y0 + r, r0, H2);
            q.a[r][0] = ll1[xe & 1][ry][ce];
            q.b[r][0] = ll1[xo & 1][ry][co];
            q.c[r][0] = ll1[2 + (xe & 1)][ry][ce];
            q.d[r][0] = ll1[2 + (xo & 1)][ry][co];
        }
    } else {
#pragma unroll
        for (int r = 0; r < R2; ++r) {
            const int Y = Y0 + r;
            const int ye = mirror(2 * Y, p2.h), yo = mirror(2 * Y + 1, p2.h);
            const int re = lds_at(ye >> 1, r0, H2), ro = lds_at(yo >> 1, r0, H2);
            const int pe = 2 * (ye & 1), po = 2 * (yo & 1);
            q.a[r][0] = ll1[pe + (xe & 1)][re][ce];
            q.b[r][0] = ll1[pe + (xo & 1)][re][co];
            q.c[r][0] = ll1[po + (xe & 1)][ro][ce];
            q.d[r][0] = ll1[po + (xo & 1)][ro][co];
        }
    }
    {
        Exchange<R2, 1, WAVES> x{reinterpret_cast<Mailbox<1, WAVES> *>(&box), wave, lane, 0};
        lift_forward<WV, SCH>(q, x);
    }
    const bool own_x = lane >= RG && lane < RG + G::FOX2 && X < p2.nqx;
    const uint32_t ob = own_x ? (uint32_t)X * (uint32_t)sizeof(TB) : kNoAccess;
    const uint32_t ol = own_x ? (uint32_t)X * (uint32_t)sizeof(TLL) : kNoAccess;
    int64_t rb = (int64_t)(r0 + wave * R2) * p2.band_pitch;   // row r0 + wr, stepped
    int64_t rl = (int64_t)(r0 + wave * R2) * p2.ll_pitch;
#pragma unroll
    for (int r = 0; r < R2; ++r, rb += p2.band_pitch, rl += p2.ll_pitch) {
        const int wr = wave * R2 + r;
        const int gy = r0 + wr;
        if (wr < RG || wr >= RG + G::FOY2 || gy >= p2.nqy) continue;   // wavefront-uniform
        store_elem<TB>(row_at<TB>(p2.hl, rb, p2.nqx), ob, q.b[r][0] * sHL);
        store_elem<TB>(row_at<TB>(p2.lh, rb, p2.nqx), ob, q.c[r][0] * sHL);
        store_elem<TB>(row_at<TB>(p2.hh, rb, p2.nqx), ob, q.d[r][0] * sHH);
        store_elem<TLL>(row_at<TLL>(p2.ll, rl, p2.nqx), ol, q.a[r][0] * sLL);
    }
}

// Levels j+1 and j of inverse window t (row-major, hd.across to a row).
template <int WV, int SCH, int ROWS, int WAVES, typename TLL, typename TB, typename TOUT, bool ODD>
__device__ __forceinline__ void inv_head_tile(const InvHead &hd, const int t,
                                              InvTileLds<ROWS, WAVES> &lds) {
    using G = WindowGeom<ROWS, WAVES>;
    using L = Wavelet<WV>;
    constexpr int RG = G::RG, H2 = G::IH2, R2 = G::IROWS2, NR1 = G::NR1;
    Mailbox<2, WAVES> &box = lds.box;     // level j+1 exchanges (smaller), then level j's
    float(&ll1)[4][H2][64] = lds.ll1;     // level j low-low as level j+1 output quads
    constexpr float down = kInvHeadroom<TLL, TB, TOUT>, up = 1.0f / down;
    const float uLL = (float)(1.0 / (L::ZL * L::ZL)) * down;
    const float uHL = (float)(1.0 / (L::ZL * L::ZH)) * down;
    const float uHH = (float)(1.0 / (L::ZH * L::ZH)) * down;
    const float uL1 = (float)(1.0 / (L::ZL * L::ZL));    // between the levels
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int ty = t / hd.across, tx = t - ty * hd.across;
    const int ox1 = tx * G::IOX1, oy1 = ty * G::IOY1;    // owned block of level j
    const int wx1 = ox1 - 2, wy1 = oy1 - RG;             // level j window origin (even)
    const int c0 = wx1 / 2 - RG, r0 = wy1 / 2 - RG;      // level j+1 window origin

    // ---- level j+1: window of 64 x H2 quads, one per lane, R2 rows per wavefront
    if (wave * R2 < H2) {
        Quads<R2, 1> q;
        inv_load_at<1, R2, TLL, TB, false>(q, hd.l2, c0 + lane, r0 + wave * R2);
#pragma unroll
        for (int r = 0; r < R2; ++r) {
            q.a[r][0] *= uLL; q.b[r][0] *= uHL; q.c[r][0] *= uHL; q.d[r][0] *= uHH;
        }
        {
            Exchange<R2, 1, WAVES> x{reinterpret_cast<Mailbox<1, WAVES> *>(&box), wave, lane, 0};
            lift_inverse<WV, SCH>(q, x);
        }
#pragma unroll
        for (int r = 0; r < R2; ++r) {
            const int wr = wave * R2 + r;
            if (wr < H2) {
                ll1[0][wr][lane] = q.a[r][0];
                ll1[1][wr][lane] = q.b[r][0];
                ll1[2][wr][lane] = q.c[r][0];
                ll1[3][wr][lane] = q.d[r][0];
            }
        }
    } else {
        idle_through_lifting<WV>();
    }
    __syncthreads();   // the low-low band is in LDS; every level j+1 exchange is done

    // ---- level j: window of 120 x NR1 quads, two per lane (lanes 60..63 idle)
    const InvParams &p1 = hd.l1;
    const int qx = wx1 + 2 * lane;
    const int qy0 = wy1 + wave * ROWS;
    Quads<ROWS, 2> q;
    inv_load_at<2, ROWS, TB, TB, ODD, false>(q, p1, qx, qy0);
    {
        // the low-low coefficient of quad (i, j) is the extended low phase
        int cx[2], px[2];
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const int xe = mirror(2 * (qx + i), p1.w) >> 1;
            cx[i] = lds_at(xe >> 1, c0, 64);
            px[i] = xe & 1;
        }
        if (qy0 >= 0 && 2 * (qy0 + ROWS) <= p1.h) {
            // all rows inside the level (wavefront-uniform): quad row gy's low
            // phase is row gy of the coarser output
#pragma unroll
            for (int r = 0; r < ROWS; ++r) {
                const int gy = qy0 + r;
                const int ry = lds_at(gy >> 1, r0, H2);
                const int py = 2 * (gy & 1);
#pragma unroll
                for (int i = 0; i < 2; ++i) q.a[r][i] = ll1[py + px[i]][ry][cx[i]];
            }
        } else {
#pragma unroll
            for (int r = 0; r < ROWS; ++r) {
                const int ye = mirror(2 * (qy0 + r), p1.h) >> 1;
                const int ry = lds_at(ye >> 1, r0, H2);
                const int py = 2 * (ye & 1);
#pragma unroll
                for (int i = 0; i < 2; ++i) q.a[r][i] = ll1[py + px[i]][ry][cx[i]];
            }
        }
    }
#pragma unroll
    for (int r = 0; r < ROWS; ++r) {
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            q.a[r][i] *= uL1; q.b[r][i] *= uHL; q.c[r][i] *= uHL; q.d[r][i] *= uHH;
        }
    }
    {
        Exchange<ROWS, 2, WAVES> x{&box, wave, lane, 0};
        lift_inverse<WV, SCH>(q, x);
    }
    const bool own_x = lane >= 1 && lane < 1 + G::IOX1 / 2;
    TOUT *out = static_cast<TOUT *>(p1.out);
    const int px0 = 2 * qx;
    const bool on = own_x && px0 < p1.w;
    int64_t ro = (int64_t)(2 * qy0) * p1.out_pitch;   // pixel row 2 (qy0 + r), stepped
#pragma unroll
    for (int r = 0; r < ROWS; ++r, ro += 2 * p1.out_pitch) {
        const int wr = wave * ROWS + r;
        const int gy = qy0 + r;
        if (wr < RG || wr >= RG + G::IOY1 || gy >= p1.nqy) continue;   // wavefront-uniform
        const float e[4] = {q.a[r][0] * up, q.b[r][0] * up, q.a[r][1] * up, q.b[r][1] * up};
        const float o[4] = {q.c[r][0] * up, q.d[r][0] * up, q.c[r][1] * up, q.d[r][1] * up};
        TOUT *r0p = out + ro;
        TOUT *r1p = r0p + p1.out_pitch;
        if (p1.stream_out) {
            store_cols<TOUT, 4, kStoreStream, false>(r0p, p1.w, px0, on, !ODD, e);
            store_cols<TOUT, 4, kStoreStream, false>(r1p, p1.w, px0, on, !ODD, o);
        } else {
            store_cols<TOUT, 4, kStoreCached, false>(r0p, p1.w, px0, on, !ODD, e);
            store_cols<TOUT, 4, kStoreCached, false>(r1p, p1.w, px0, on, !ODD, o);
        }
    }
}

// A window of one image of several. ODD: the launch has images whose rows may
// start at odd halves; the others take the word path in it all the same.
template <int WV, int SCH, int ROWS, int WAVES, typename TIN, typename TLL, typename TB, bool ODD>
__device__ __forceinline__ void fwd_image_window(const FwdHead &hd, const int t,
                                                 FwdTileLds<ROWS, WAVES> &lds) {
    if (ODD && odd_rows(hd))   // workgroup-uniform
        fwd_head_tile<WV, SCH, ROWS, WAVES, TIN, TLL, TB, ODD>(hd, t, lds);
    else
        fwd_head_tile<WV, SCH, ROWS, WAVES, TIN, TLL, TB, false>(hd, t, lds);
}
template <int WV, int SCH, int ROWS, int WAVES, typename TLL, typename TB, typename TOUT, bool ODD>
__device__ __forceinline__ void inv_image_window(const InvHead &hd, const int t,
                                                 InvTileLds<ROWS, WAVES> &lds) {
    if (ODD && odd_rows(hd))   // workgroup-uniform
        inv_head_tile<WV, SCH, ROWS, WAVES, TLL, TB, TOUT, ODD>(hd, t, lds);
    else
        inv_head_tile<WV, SCH, ROWS, WAVES, TLL, TB, TOUT, false>(hd, t, lds);
}

// One workgroup per tile of one image.
template <int WV, int SCH, int ROWS, int WAVES, typename TIN, typename TLL, typename TB, bool ODD>
__global__ __launch_bounds__(64 * WAVES, (kFwdHeadWavesPerSimd<SCH, WAVES, TIN>)) void fwd_head_tile_kernel(
    FwdHead hd) {
    __shared__ FwdTileLds<ROWS, WAVES> lds;
    fwd_head_tile<WV, SCH, ROWS, WAVES, TIN, TLL, TB, ODD>(hd, block_tile(), lds);
}

template <int WV, int SCH, int ROWS, int WAVES, typename TLL, typename TB, typename TOUT, bool ODD>
__global__ __launch_bounds__(64 * WAVES, kInvHeadWavesPerSimd<WAVES>) void inv_head_tile_kernel(InvHead hd) {
    __shared__ InvTileLds<ROWS, WAVES> lds;
    inv_head_tile<WV, SCH, ROWS, WAVES, TLL, TB, TOUT, ODD>(hd, block_tile(), lds);
}

// Heads of a planned batch: the tiles of every image in one launch, each
// image's parameters in the device copy of the plan. A workgroup walks the
// tiles t = its id, id + gridDim.x, ... below `total` (several when the grid is
// capped at the resident workgroups), with a barrier between tiles, which
// share the LDS.
template <int WV, int SCH, int ROWS, int WAVES, typename TIN, typename TLL, typename TB, bool ODD>
__global__ __launch_bounds__(64 * WAVES, kTableHeadWavesPerSimd<WAVES>) void fwd_head_tile_table_kernel(
    TableLaunch<FwdHead> tl) {
    __shared__ FwdTileLds<ROWS, WAVES> lds;
    for (int t = block_tile(); t < tl.total; t += gridDim.x) {
        const int i = load_uniform(tl.img + t);
        const FwdHead hd = load_uniform(tl.params + i);
        fwd_image_window<WV, SCH, ROWS, WAVES, TIN, TLL, TB, ODD>(hd, t - load_uniform(tl.start + i), lds);
        __syncthreads();
    }
}

template <int WV, int SCH, int ROWS, int WAVES, typename TLL, typename TB, typename TOUT, bool ODD>
__global__ __launch_bounds__(64 * WAVES, kTableHeadWavesPerSimd<WAVES>) void inv_head_tile_table_kernel(
    TableLaunch<InvHead> tl) {
    __shared__ InvTileLds<ROWS, WAVES> lds;
    for (int t = block_tile(); t < tl.total; t += gridDim.x) {
        const int i = load_uniform(tl.img + t);
        const InvHead hd = load_uniform(tl.params + i);
        inv_image_window<WV, SCH, ROWS, WAVES, TLL, TB, TOUT, ODD>(hd, t - load_uniform(tl.start + i), lds);
        __syncthreads();
    }
}

// Heads of independent images in one launch, one workgroup per tile.
template <int WV, int SCH, int ROWS, int WAVES, typename TIN, typename TLL, typename TB, bool ODD>
__global__ __launch_bounds__(64 * WAVES, kTableHeadWavesPerSimd<WAVES>) void fwd_head_tile_batch_kernel(
    FwdHeadBatch bt) {
    __shared__ FwdTileLds<ROWS, WAVES> lds;
    const int t = block_tile();
    const int i = batch_image(bt, t);
    fwd_image_window<WV, SCH, ROWS, WAVES, TIN, TLL, TB, ODD>(bt.h[i], t - bt.tile_start[i], lds);
}

template <int WV, int SCH, int ROWS, int WAVES, typename TLL, typename TB, typename TOUT, bool ODD>
__global__ __launch_bounds__(64 * WAVES, kTableHeadWavesPerSimd<WAVES>) void inv_head_tile_batch_kernel(
    InvHeadBatch bt) {
    __shared__ InvTileLds<ROWS, WAVES> lds;
    const int t = block_tile();
    const int i = batch_image(bt, t);
    inv_image_window<WV, SCH, ROWS, WAVES, TLL, TB, TOUT, ODD>(bt.h[i], t - bt.tile_start[i], lds);
}

}  // namespace dwt2
