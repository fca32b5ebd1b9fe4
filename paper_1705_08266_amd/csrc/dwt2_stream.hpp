// Rows streamed through the lifting: the register pipelines of the fused
// finest levels.
//
// A wavefront sweeps down a strip of quad columns, one quad row after the
// other. Each lifting pair is one stage of a pipeline: it holds the row that
// waits for the row below it (T_P reads the lower neighbours) and what S_U
// needs of the row above; pushing row r in emits row r - 1 finished. Stages
// follow each other without leaving the registers, so a row is read once,
// nothing goes through LDS and no wavefront needs another's data (the barrier
// per row pair that the sweeps pass only keeps neighbouring strips together).
//
// Arithmetic per quad is that of the register-tile steps (dwt2_device.hpp),
// term by term, so the results are the same bits.
//
// Image edges. A missing neighbour is the quad's own value (the symmetric
// extension as the steps see it, see add_right): `first` / `last` mark the
// lane whose quad is the level's first / last column, `top` / `bottom` the
// row. Only wavefronts at a left or right (EX), upper or lower (EY) edge of the
// image compute with the marks; columns and rows outside the level are never
// looked at.
#pragma once

#include "dwt2_device.hpp"

namespace dwt2 {

// ---- row access of a strip -------------------------------------------------------
// How rows are addressed.
//   ROWS_NEAR: one resource, based at the segment's first row, reaches every row
//     through a 32-bit row offset that steps with the rows; lanes that must not
//     access use kNoAccess, beyond any row.
//   ROWS_ODD: the same for 2-byte elements whose rows are not aligned to the
//     vectors. Loads take the whole words that hold the elements and shift
//     them into place by the row's misalignment, which all lanes share (an
//     element at a time: 4 loads for one); stores go by halves and words where
//     a row is not word aligned.
//   ROWS_FAR: rows may be too far apart for 32 bits: each gets its own resource.
//     2-byte elements are taken as in ROWS_ODD.
enum : int { ROWS_NEAR = 0, ROWS_ODD = 1, ROWS_FAR = 2 };
constexpr uint32_t kSpan = 0x7ffffff0u;

template <int NW> struct Words { typedef uint32_t type __attribute__((ext_vector_type(NW))); };
template <> struct Words<1> { typedef uint32_t type; };

// N consecutive elements of T as the raw words of their load. The words stay
// one value (not an array of scalars) from the load to their use rows later.
template <typename T, int N, int MODE>
struct Raw {
    static constexpr bool HALF = sizeof(T) == 2;
    static constexpr bool SHIFT = HALF && N > 1 && MODE != ROWS_NEAR;
    static constexpr int NW = !HALF ? N : N == 1 ? 1 : N / 2 + (SHIFT ? 1 : 0);
    typename Words<NW>::type w;
    uint32_t shift;   // bits; wavefront-uniform

    // `odd`: the row starts at the upper half of the word at `soff`.
    __device__ __forceinline__ void load(rsrc_t r, uint32_t off, uint32_t soff, bool odd) {
        shift = odd ? 16u : 0u;
        if constexpr (SHIFT) {   // only lane offsets are checked against the buffer's end
            off += soff;
            soff = 0;
        }
        if constexpr (HALF && N == 1) {
            w = (uint32_t)(uint16_t)__builtin_amdgcn_raw_buffer_load_b16(
                r, (int)off, (int)(soff + (odd ? 2u : 0u)), 0);
        } else if constexpr (NW == 1) {
            w = __builtin_amdgcn_raw_buffer_load_b32(r, (int)off, (int)soff, 0);
        } else if constexpr (NW == 2) {
            w = __builtin_amdgcn_raw_buffer_load_b64(r, (int)off, (int)soff, 0);
        } else if constexpr (NW == 3) {
            w = __builtin_amdgcn_raw_buffer_load_b96(r, (int)off, (int)soff, 0);
        } else {
            static_assert(NW == 4, "access width");
            w = __builtin_amdgcn_raw_buffer_load_b128(r, (int)off, (int)soff, 0);
        }
    }
    __device__ __forceinline__ float get(int i) const {
        if constexpr (!HALF) {
            if constexpr (NW == 1) return __uint_as_float(w);
            else return __uint_as_float(w[i]);
        } else if constexpr (N == 1) {
            return Storage<T>::decode(w);
        } else {
            uint32_t v;
            if constexpr (SHIFT) v = __builtin_amdgcn_alignbit(w[i / 2 + 1], w[i / 2], shift);
            else if constexpr (NW == 1) v = w;
            else v = w[i / 2];
            return Storage<T>::decode((v >> (16 * (i & 1))) & 0xffffu);
        }
    }
};

// Rows of one buffer as a strip sees them, from row `row0` on.
template <typename T, int MODE>
struct RowsOf {
    static constexpr bool HALF = sizeof(T) == 2;
    static constexpr bool ODD = HALF && MODE != ROWS_NEAR;
    const T *base;       // of row 0 (ROWS_FAR), else of row row0
    int64_t pitch;
    int row0, n;
    uint32_t row_bytes, step, odd0, span;

    __device__ __forceinline__ RowsOf(const void *b, int64_t pitch_, int n_, int w, int row0_)
        : base(static_cast<const T *>(b)), pitch(pitch_), row0(row0_), n(n_),
          row_bytes((uint32_t)w * (uint32_t)sizeof(T)),
          step((uint32_t)(pitch_ * (int64_t)sizeof(T))), odd0(0), span(kSpan) {
        if constexpr (MODE != ROWS_FAR) base += (int64_t)row0 * pitch;
        if constexpr (MODE == ROWS_ODD && HALF) {
            odd0 = (uint32_t)((uintptr_t)base & 2u);
            base = reinterpret_cast<const T *>((uintptr_t)base & ~(uintptr_t)3);
            // up to the word that holds the last element: a lane's last word may
            // lie past it
            const int64_t end = (int64_t)(n - 1 - row0) * pitch * (int64_t)sizeof(T) + row_bytes + odd0;
            span = (uint32_t)min((end + 3) & ~(int64_t)3, (int64_t)kSpan);
        }
    }
    // The resource and word-aligned offset of row `row`, and whether it starts at
    // the upper half of a word; s is the row's stepped offset.
    __device__ __forceinline__ rsrc_t place(int row, uint32_t s, uint32_t &soff, bool &odd) const {
        odd = false;
        if constexpr (MODE == ROWS_FAR) {
            uintptr_t a = (uintptr_t)(base + (int64_t)min(max(row, 0), n - 1) * pitch);
            soff = 0;
            if constexpr (HALF) odd = (a & 2u) != 0;
            if constexpr (HALF) a &= ~(uintptr_t)3;
            return make_rsrc(reinterpret_cast<const void *>(a), (row_bytes + (odd ? 2u : 0u) + 3u) & ~3u);
        } else if constexpr (MODE == ROWS_ODD && HALF) {
            odd = ((odd0 + s) & 2u) != 0;
            soff = (odd0 + s) & ~3u;
            return make_rsrc(base, span);
        } else {
            soff = s;
            return make_rsrc(base, kSpan);
        }
    }
    // Loads N elements at byte `off` of row `row`: EY: rows outside the level
    // stand for its first or last.
    template <bool EY, int N>
    __device__ __forceinline__ void load(Raw<T, N, MODE> &v, int row, uint32_t off, uint32_t s) const {
        if constexpr (EY && MODE != ROWS_FAR) s = (uint32_t)(min(max(row, 0), n - 1) - row0) * step;
        uint32_t soff;
        bool odd;
        const rsrc_t r = place(row, s, soff, odd);
        v.load(r, off, soff, odd);
    }
    // Stores N elements at byte `off` of row `row`.
    template <int N, int POLICY = kStoreCached>
    __device__ __forceinline__ void store(int row, uint32_t off, uint32_t s, const float (&v)[N]) const {
        uint32_t soff;
        bool odd;
        const rsrc_t r = place(row, s, soff, odd);
        constexpr int NW = N * (int)sizeof(T) / 4;
        uint32_t w[NW > 0 ? NW : 1];
        if constexpr (!HALF) {
#pragma unroll
            for (int i = 0; i < N; ++i) w[i] = __float_as_uint(v[i]);
        } else if constexpr (N == 1) {
            w[0] = bits_of<T>(from_float<T>(v[0]));
        } else {
#pragma unroll
            for (int i = 0; i < N; i += 2) w[i / 2] = pack2<T>(v[i], v[i + 1]);
        }
        if constexpr (HALF && N == 1) {
            __builtin_amdgcn_raw_buffer_store_b16((unsigned short)w[0], r, (int)off,
                                                  (int)(soff + (odd ? 2u : 0u)), POLICY);
            return;
        } else {
            if (ODD && odd) {   // wavefront-uniform: the halves at the ends, words between
                __builtin_amdgcn_raw_buffer_store_b16((unsigned short)w[0], r, (int)(off + 2u),
                                                      (int)soff, POLICY);
#pragma unroll
                for (int i = 1; i < NW; ++i)
                    __builtin_amdgcn_raw_buffer_store_b32(
                        __builtin_amdgcn_alignbit(w[i], w[i - 1], 16), r, (int)(off + 4u * i),
                        (int)soff, POLICY);
                __builtin_amdgcn_raw_buffer_store_b16((unsigned short)(w[NW - 1] >> 16), r,
                                                      (int)(off + 4u * NW), (int)soff, POLICY);
                return;
            }
            if constexpr (NW == 1) {
                __builtin_amdgcn_raw_buffer_store_b32(w[0], r, (int)off, (int)soff, POLICY);
            } else if constexpr (NW == 2) {
                u32x2 x; x.x = w[0]; x.y = w[1];
                __builtin_amdgcn_raw_buffer_store_b64(x, r, (int)off, (int)soff, POLICY);
            } else {
                static_assert(NW == 4, "access width");
                u32x4 x; x.x = w[0]; x.y = w[1]; x.z = w[2]; x.w = w[3];
                // the row offset goes into the lane offset: a 16-byte store whose
                // row offset is a scalar register still reads its data when the
                // next instruction writes those registers, and the compiler puts
                // the wait state between the two only where there is no scalar
                // offset (16384^2 FP32 inverse: 0.04% of the pixels wrong)
                __builtin_amdgcn_raw_buffer_store_b128(x, r, (int)(off + soff), 0, POLICY);
            }
        }
    }
};

// n stores that the hardware drops. Loads and stores complete in order, and the
// compiler waits for a load by the number of accesses issued after it; on
// entry to a row loop it takes the smaller of the numbers before the loop and
// around it. Issued between the first loads, these make the two equal, so that
// the loop's first row does not wait for the rows after it.
__device__ __forceinline__ void pad_stores(int n) {
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int k = 0; k < n; ++k)
        __builtin_amdgcn_raw_buffer_store_b32(0u, make_rsrc(nullptr, 0u), (int)kNoAccess, 0, 0);
    __builtin_amdgcn_sched_barrier(0);
}

// ---- pipeline ---------------------------------------------------------------------
// One quad row of a lane: QPL consecutive quads.
template <int QPL>
struct Line {
    float a[QPL], b[QPL], c[QPL], d[QPL];
};

struct ColMarks {
    bool first, last;   // the lane holds the level's first / last column
};

template <bool EX, int QPL>
__device__ __forceinline__ void sum_right(const float (&x)[QPL], float (&s)[QPL], ColMarks m) {
    float xr = from_right(x[0]);
    if constexpr (EX) xr = m.last ? x[QPL - 1] : xr;
#pragma unroll
    for (int i = 0; i < QPL; ++i) s[i] = x[i] + ((i + 1 < QPL) ? x[(i + 1 < QPL) ? i + 1 : i] : xr);
}
template <bool EX, int QPL>
__device__ __forceinline__ void sum_left(const float (&x)[QPL], float (&s)[QPL], ColMarks m) {
    float xl = from_left(x[QPL - 1]);
    if constexpr (EX) xl = m.first ? x[0] : xl;
#pragma unroll
    for (int i = 0; i < QPL; ++i) s[i] = x[i] + ((i > 0) ? x[(i > 0) ? i - 1 : i] : xl);
}

// One forward lifting pair (T_P, then S_U).
//   push(x, bottom, top): x is row r; emits row r - 1 in x. bottom (top): row
//   r - 1 is the level's last (first) row.
template <int SCH, int QPL, bool EX, bool EY>
struct FwdStage {
    Line<QPL> y;                // the waiting row: b after T_P (separable: d after T_P^H too)
    float pc[QPL], pd[QPL];     // of the row above y: what S_U^V adds

    __device__ __forceinline__ void push(Line<QPL> &x, float p, float u, ColMarks m, bool bottom,
                                         bool top) {
        float s[QPL], sc[QPL];
        Line<QPL> z = y;        // becomes the finished row r - 1
        // row r, on arrival: the horizontal part of T_P
        sum_right<EX>(x.a, s, m);
        if constexpr (SCH != NONSEP) sum_right<EX>(x.c, sc, m);
#pragma unroll
        for (int i = 0; i < QPL; ++i) {
            x.b[i] = fmaf(p, s[i], x.b[i]);
            if constexpr (SCH != NONSEP) x.d[i] = fmaf(p, sc[i], x.d[i]);
        }
        // row r - 1: the rest of T_P
        if constexpr (SCH == NONSEP) sum_right<EX>(z.c, sc, m);
        float c[QPL];
#pragma unroll
        for (int i = 0; i < QPL; ++i) {
            float xa = x.a[i], xb = x.b[i];
            if constexpr (EY) {
                xa = bottom ? z.a[i] : xa;
                xb = bottom ? z.b[i] : xb;
            }
            c[i] = fmaf(p, z.a[i] + xa, z.c[i]);
            if constexpr (SCH == NONSEP) z.d[i] = fmaf(p, z.b[i] + xb, fmaf(p, sc[i], z.d[i]));
            else z.d[i] = fmaf(p, z.b[i] + xb, z.d[i]);
        }
        // row r - 1: S_U
        if constexpr (SCH == NONSEP) {
            float sd[QPL], sb[QPL];
            sum_left<EX>(z.d, sd, m);
#pragma unroll
            for (int i = 0; i < QPL; ++i) {
                if constexpr (EY) {
                    pc[i] = top ? c[i] : pc[i];
                    pd[i] = top ? z.d[i] : pd[i];
                }
                z.b[i] = fmaf(u, z.d[i] + pd[i], z.b[i]);
            }
            sum_left<EX>(z.b, sb, m);
#pragma unroll
            for (int i = 0; i < QPL; ++i) {
                z.a[i] = fmaf(u, sb[i] + (c[i] + pc[i]), z.a[i]);
                z.c[i] = fmaf(u, sd[i], c[i]);
                pc[i] = c[i];
                pd[i] = z.d[i];
            }
        } else {
            float sd[QPL], sb[QPL];
            sum_left<EX>(z.b, sb, m);
            sum_left<EX>(z.d, sd, m);
#pragma unroll
            for (int i = 0; i < QPL; ++i) {
                z.a[i] = fmaf(u, sb[i], z.a[i]);
                z.c[i] = fmaf(u, sd[i], c[i]);
                if constexpr (EY) {
                    pc[i] = top ? z.c[i] : pc[i];
                    pd[i] = top ? z.d[i] : pd[i];
                }
                z.a[i] = fmaf(u, z.c[i] + pc[i], z.a[i]);
                z.b[i] = fmaf(u, z.d[i] + pd[i], z.b[i]);
                pc[i] = z.c[i];
                pd[i] = z.d[i];
            }
        }
        y = x;
        x = z;
    }
};

// One inverse lifting pair (S_U undone, then T_P; p and u negated by the
// caller). push(x, top, bottom): x is row r, top: r is the level's first row;
// emits row r - 1, bottom: that is the level's last.
template <int SCH, int QPL, bool EX, bool EY>
struct InvStage {
    Line<QPL> y;                // the waiting row: S_U undone (non-separable: b with T_P undone)
    float pc[QPL], pd[QPL];     // c, d of the row above the next one, as they came

    __device__ __forceinline__ void push(Line<QPL> &x, float p, float u, ColMarks m, bool top,
                                         bool bottom) {
        float sd[QPL], sb[QPL], s[QPL], sc[QPL];
        Line<QPL> z = y;
        if constexpr (EY) {
#pragma unroll
            for (int i = 0; i < QPL; ++i) {
                pc[i] = top ? x.c[i] : pc[i];
                pd[i] = top ? x.d[i] : pd[i];
            }
        }
        // row r: S_U
        if constexpr (SCH == NONSEP) {
            sum_left<EX>(x.d, sd, m);
#pragma unroll
            for (int i = 0; i < QPL; ++i) x.b[i] = fmaf(u, x.d[i] + pd[i], x.b[i]);
            sum_left<EX>(x.b, sb, m);
#pragma unroll
            for (int i = 0; i < QPL; ++i) {
                const float c = x.c[i];
                x.a[i] = fmaf(u, sb[i] + (c + pc[i]), x.a[i]);
                x.c[i] = fmaf(u, sd[i], c);
                pc[i] = c;
                pd[i] = x.d[i];
            }
            // its b is done with the row's own a
            sum_right<EX>(x.a, s, m);
#pragma unroll
            for (int i = 0; i < QPL; ++i) x.b[i] = fmaf(p, s[i], x.b[i]);
        } else {
#pragma unroll
            for (int i = 0; i < QPL; ++i) {
                x.a[i] = fmaf(u, x.c[i] + pc[i], x.a[i]);
                x.b[i] = fmaf(u, x.d[i] + pd[i], x.b[i]);
                pc[i] = x.c[i];
                pd[i] = x.d[i];
            }
            sum_left<EX>(x.b, sb, m);
            sum_left<EX>(x.d, sd, m);
#pragma unroll
            for (int i = 0; i < QPL; ++i) {
                x.a[i] = fmaf(u, sb[i], x.a[i]);
                x.c[i] = fmaf(u, sd[i], x.c[i]);
            }
        }
        // row r - 1: T_P
        if constexpr (SCH == NONSEP) sum_right<EX>(z.c, sc, m);
#pragma unroll
        for (int i = 0; i < QPL; ++i) {
            float xa = x.a[i], xb = x.b[i];
            if constexpr (EY) {
                xa = bottom ? z.a[i] : xa;
                xb = bottom ? z.b[i] : xb;
            }
            if constexpr (SCH == NONSEP) z.d[i] = fmaf(p, z.b[i] + xb, fmaf(p, sc[i], z.d[i]));
            else z.d[i] = fmaf(p, z.b[i] + xb, z.d[i]);
            z.c[i] = fmaf(p, z.a[i] + xa, z.c[i]);
        }
        if constexpr (SCH != NONSEP) {
            sum_right<EX>(z.a, s, m);
            sum_right<EX>(z.c, sc, m);
#pragma unroll
            for (int i = 0; i < QPL; ++i) {
                z.b[i] = fmaf(p, s[i], z.b[i]);
                z.d[i] = fmaf(p, sc[i], z.d[i]);
            }
        }
        y = x;
        x = z;
    }
};

// All lifting pairs of one level. push(x, r, n): x is row r of n; emits row
// r - NPAIRS.
template <int WV, int SCH, int QPL, bool EX, bool EY>
struct FwdRows {
    static constexpr int NP = Wavelet<WV>::NPAIRS;
    FwdStage<SCH, QPL, EX, EY> s0;
    FwdStage<SCH, QPL, EX, EY> s1;   // 9/7 only
    __device__ __forceinline__ void push(Line<QPL> &x, int r, int n, ColMarks m) {
        using L = Wavelet<WV>;
        s0.push(x, (float)L::p(0), (float)L::u(0), m, r - 1 == n - 1, r - 1 == 0);
        if constexpr (NP == 2)
            s1.push(x, (float)L::p(1), (float)L::u(1), m, r - 2 == n - 1, r - 2 == 0);
    }
};
template <int WV, int SCH, int QPL, bool EX, bool EY>
struct InvRows {
    static constexpr int NP = Wavelet<WV>::NPAIRS;
    InvStage<SCH, QPL, EX, EY> st[NP];
    __device__ __forceinline__ void push(Line<QPL> &x, int r, int n, ColMarks m) {
        using L = Wavelet<WV>;
#pragma unroll
        for (int k = 0; k < NP; ++k)
            st[k].push(x, -(float)L::p(NP - 1 - k), -(float)L::u(NP - 1 - k), m, r - k == 0,
                       r - k - 1 == n - 1);
    }
};

}  // namespace dwt2
