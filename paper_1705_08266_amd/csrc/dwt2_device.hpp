// Device-side building blocks of the 2-D lifting DWT for gfx950 (CDNA4).
//
// Data layout in registers. A workgroup owns a window of quads: 64 lanes per
// wavefront along x, each lane holding QPL consecutive quads of a quad row,
// and ROWS quad rows per lane; WAVES wavefronts are stacked along y. A quad is
// the 2x2 polyphase block (a, b, c, d) = (x[2j][2i], x[2j][2i+1],
// x[2j+1][2i], x[2j+1][2i+1]), the paper's components 1..4 (Sec. 2).
//
// Neighbour exchange. Horizontal neighbours of the first/last quad of a lane
// come from the adjacent lane through DPP wavefront shifts (no LDS, no
// barrier); vertical neighbours inside a lane's rows are registers; the rows
// on the boundary between two wavefronts go through a small double-buffered
// LDS mailbox, one workgroup barrier per exchange. Window edges read
// don't-care values; the lifting halo around the written centre absorbs them.
#pragma once

#include <hip/hip_runtime.h>
#include <hip/hip_fp16.h>
#include <stdint.h>

#include <type_traits>

// A product and a sum are never fused unless fmaf says so: the same lifting
// inlined into different kernels has to round alike.
#pragma clang fp contract(off)

namespace dwt2 {

enum : int { CDF97 = 0, CDF53 = 1 };
// NONSEP_LDS and SEP_LDS are the same schemes with every neighbour exchange
// going through LDS and a workgroup barrier, horizontal ones included (the
// paper's local-memory design), instead of DPP lane shifts.
enum : int { NONSEP = 0, SEP = 1, NONSEP_LDS = 2, SEP_LDS = 3 };
enum : int { DT_F32 = 0, DT_F16 = 1, DT_BF16 = 2 };

// ---- lifting constants ------------------------------------------------------
// CDF 9/7: two pairs (alpha, beta), (gamma, delta) and the scaling K; CDF 5/3:
// one pair (-1/2, 1/4). Predicts P(z) = p (1 + z), updates U(z) = u (1 + 1/z).
// Unit-gain scaling: low phase * 1/K, high phase * K/2 (5/3: 1 and 1/2).
template <int WV> struct Wavelet;

template <> struct Wavelet<CDF97> {
    static constexpr int NPAIRS = 2;
    static constexpr double K = 1.230174104914001;
    __host__ __device__ static constexpr double p(int k) { return k == 0 ? -1.586134342059924 : 0.882911075530934; }
    __host__ __device__ static constexpr double u(int k) { return k == 0 ? -0.052980118572961 : 0.443506852043971; }
    static constexpr double ZL = 1.0 / K;
    static constexpr double ZH = K / 2.0;
};

template <> struct Wavelet<CDF53> {
    static constexpr int NPAIRS = 1;
    __host__ __device__ static constexpr double p(int) { return -0.5; }
    __host__ __device__ static constexpr double u(int) { return 0.25; }
    static constexpr double ZL = 1.0;
    static constexpr double ZH = 0.5;
};

// ---- storage types ----------------------------------------------------------
struct bf16_t { uint16_t bits; };

template <typename T> struct Storage;
template <> struct Storage<float> {
    static constexpr int code = DT_F32;
    __device__ static float decode(uint32_t v) { return __uint_as_float(v); }
};
template <> struct Storage<__half> {
    static constexpr int code = DT_F16;
    __device__ static float decode(uint32_t v) {
        return __half2float(__ushort_as_half((unsigned short)v));
    }
};
template <> struct Storage<bf16_t> {
    static constexpr int code = DT_BF16;
    __device__ static float decode(uint32_t v) { return __uint_as_float(v << 16); }
};

// Headroom of the lifting. Its steps add up to four neighbours before they
// multiply, and such a sum may exceed FLT_MAX where every value of the transform
// is in range (a 5/3 image of 1.8e38, 9/7 stripes of 2e37). So values are
// scaled by 2^-2 on the way in and back on the way out, and a step overflows only
// where its result does. A power of two changes no bit of a result beyond
// 2^-124. Halves end at 65504, whose sums are far from the limit: where nothing
// but halves comes in, or goes out, the factor is 1. Elsewhere a forward
// multiplies its pixels and an inverse its results once more; the factors at
// the other end are there already. Between fused levels the low-low band stays
// scaled: one that exceeds FLT_MAX itself is infinite only where it is stored.
template <typename... T>
constexpr bool kAllHalf = (std::is_same<T, __half>::value && ...);
template <typename TIN>
constexpr float kFwdHeadroom = kAllHalf<TIN> ? 1.0f : 0.25f;
template <typename TLL, typename TB, typename TOUT>
constexpr float kInvHeadroom = kAllHalf<TOUT> || kAllHalf<TLL, TB> ? 1.0f : 0.25f;

__device__ __forceinline__ float to_float(float v) { return v; }
__device__ __forceinline__ float to_float(__half v) { return __half2float(v); }
__device__ __forceinline__ float to_float(bf16_t v) { return __uint_as_float((uint32_t)v.bits << 16); }

// Round-to-nearest-even conversions from FP32.
template <typename T> __device__ __forceinline__ T from_float(float v);
template <> __device__ __forceinline__ float from_float<float>(float v) { return v; }
// The value is pinned in an FP32 register first: otherwise the compiler may
// fuse the multiply that produced it into an FMA with FP16 output (one
// rounding instead of FP32-then-FP16), and results would depend on the
// kernel configuration.
template <> __device__ __forceinline__ __half from_float<__half>(float v) {
    asm volatile("" : "+v"(v));
    return __float2half_rn(v);
}
// A NaN stays a quiet NaN with its sign.
template <> __device__ __forceinline__ bf16_t from_float<bf16_t>(float v) {
    bf16_t r;
    r.bits = __builtin_bit_cast(uint16_t, (__bf16)v);
    return r;
}

template <typename T> __device__ __forceinline__ uint32_t bits_of(T v);
template <> __device__ __forceinline__ uint32_t bits_of<float>(float v) { return __float_as_uint(v); }
template <> __device__ __forceinline__ uint32_t bits_of<__half>(__half v) { return (uint32_t)__half_as_ushort(v); }
template <> __device__ __forceinline__ uint32_t bits_of<bf16_t>(bf16_t v) { return v.bits; }

// Two values as one word of 2-byte elements (lo in the low half), by the
// hardware's packed conversion: the same bits as from_float for every input
// (all 2^32 compared), in one instruction where two conversions and their
// packing take three (FP16) and rounding in integers with its NaN test took
// about a dozen (BF16). The fused heads are bound by the instructions they
// issue at these sizes: 2048^2 BF16 forward 15.4 -> 13.3 us, 4096^2 27.4 -> 24.9.
template <typename T> __device__ __forceinline__ uint32_t pack2(float lo, float hi);
template <> __device__ __forceinline__ uint32_t pack2<__half>(float lo, float hi) {
    typedef float f32x2 __attribute__((ext_vector_type(2)));
    typedef _Float16 f16x2 __attribute__((ext_vector_type(2)));
    asm("" : "+v"(lo), "+v"(hi));   // FP32 values first, as in from_float
    const f32x2 v = {lo, hi};
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, f16x2));
}
template <> __device__ __forceinline__ uint32_t pack2<bf16_t>(float lo, float hi) {
    typedef float f32x2 __attribute__((ext_vector_type(2)));
    typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
    const f32x2 v = {lo, hi};
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2));
}

// ---- vector row access through buffer resources ---------------------------------
// A row of a 2-D buffer is described by a wave-uniform buffer resource (base
// pointer and byte length); each lane addresses it with a 32-bit byte offset.
// The hardware checks every access against the length: reads past the end
// return zero and writes past the end are dropped.
using rsrc_t = __amdgpu_buffer_rsrc_t;
constexpr int kRsrcWord3 = 0x00020000;   // raw (untyped) buffer, gfx9 family

__device__ __forceinline__ rsrc_t make_rsrc(const void *base, uint32_t bytes) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(base), (short)0, (int)bytes,
                                             kRsrcWord3);
}

// Cache policy of a buffer store (the instruction's cache-policy operand).
// kStoreStream sets the non-temporal bit: the written lines go out to memory
// without being kept in the caches for reuse, for output that no later step
// of the transform reads.
constexpr int kStoreCached = 0, kStoreStream = 2;

typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x3 __attribute__((ext_vector_type(3)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

// Raw 32-bit words of an access of W words.
template <int W>
__device__ __forceinline__ void buf_load_words(rsrc_t r, uint32_t off, uint32_t (&w)[W]) {
    static_assert(W >= 1 && W <= 8, "access width");
    // kNoAccess plus the width stays beyond any row
#pragma unroll
    for (int h = 0; h < W / 4; ++h) {
        u32x4 v = __builtin_amdgcn_raw_buffer_load_b128(r, (int)(off + 16u * h), 0, 0);
        w[4 * h] = v.x; w[4 * h + 1] = v.y; w[4 * h + 2] = v.z; w[4 * h + 3] = v.w;
    }
    constexpr int B = W & ~3;
    if constexpr (W - B == 1) {
        w[B] = __builtin_amdgcn_raw_buffer_load_b32(r, (int)(off + 4u * B), 0, 0);
    } else if constexpr (W - B == 2) {
        u32x2 v = __builtin_amdgcn_raw_buffer_load_b64(r, (int)(off + 4u * B), 0, 0);
        w[B] = v.x; w[B + 1] = v.y;
    } else if constexpr (W - B == 3) {
        u32x3 v = __builtin_amdgcn_raw_buffer_load_b96(r, (int)(off + 4u * B), 0, 0);
        w[B] = v.x; w[B + 1] = v.y; w[B + 2] = v.z;
    }
}

template <int W, int POLICY = kStoreCached>
__device__ __forceinline__ void buf_store_words(rsrc_t r, uint32_t off, const uint32_t (&w)[W]) {
    static_assert(W == 1 || W == 2 || W == 4 || W == 8, "access width");
    if constexpr (W == 1) {
        __builtin_amdgcn_raw_buffer_store_b32(w[0], r, (int)off, 0, POLICY);
    } else if constexpr (W == 2) {
        u32x2 v; v.x = w[0]; v.y = w[1];
        __builtin_amdgcn_raw_buffer_store_b64(v, r, (int)off, 0, POLICY);
    } else {
#pragma unroll
        for (int h = 0; h < W / 4; ++h) {
            u32x4 v; v.x = w[4 * h]; v.y = w[4 * h + 1]; v.z = w[4 * h + 2]; v.w = w[4 * h + 3];
            __builtin_amdgcn_raw_buffer_store_b128(v, r, (int)(off + 16u * h), 0, POLICY);
        }
    }
}

// One element of type T at byte offset `off` (reads past the end give 0).
template <typename T>
__device__ __forceinline__ float load_elem(rsrc_t r, uint32_t off) {
    if constexpr (sizeof(T) == 4) {
        return __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(r, (int)off, 0, 0));
    } else {
        return Storage<T>::decode((uint32_t)__builtin_amdgcn_raw_buffer_load_b16(r, (int)off, 0, 0));
    }
}

template <typename T>
__device__ __forceinline__ void store_elem(rsrc_t r, uint32_t off, float v) {
    if constexpr (sizeof(T) == 4) {
        __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(v), r, (int)off, 0, 0);
    } else {
        __builtin_amdgcn_raw_buffer_store_b16((unsigned short)bits_of<T>(from_float<T>(v)), r,
                                              (int)off, 0, 0);
    }
}

// A byte offset that every buffer resource of this library rejects: rows
// are shorter than 2 GiB, so a store at this offset is dropped.
constexpr uint32_t kNoAccess = 0x80000000u;

// N consecutive elements of type T (2 to 32 bytes) at byte offset `off`.
template <typename T, int N>
__device__ __forceinline__ void load_vec(rsrc_t r, uint32_t off, float (&out)[N]) {
    constexpr int BYTES = N * (int)sizeof(T);
    if constexpr (BYTES == 2) {
        out[0] = load_elem<T>(r, off);
    } else {
        static_assert(BYTES % 4 == 0, "whole words");
        uint32_t w[BYTES / 4];
        buf_load_words<BYTES / 4>(r, off, w);
        if constexpr (sizeof(T) == 4) {
#pragma unroll
            for (int e = 0; e < N; ++e) out[e] = __uint_as_float(w[e]);
        } else {
#pragma unroll
            for (int e = 0; e < N; ++e)
                out[e] = Storage<T>::decode((w[e / 2] >> (16 * (e & 1))) & 0xffffu);
        }
    }
}

template <typename T, int N, int POLICY = kStoreCached>
__device__ __forceinline__ void store_vec(rsrc_t r, uint32_t off, const float (&in)[N]) {
    constexpr int BYTES = N * (int)sizeof(T);
    if constexpr (BYTES == 2) {
        store_elem<T>(r, off, in[0]);
    } else {
        static_assert(BYTES % 4 == 0, "whole words");
        uint32_t w[BYTES / 4];
        if constexpr (sizeof(T) == 4) {
#pragma unroll
            for (int e = 0; e < N; ++e) w[e] = __float_as_uint(in[e]);
        } else {
#pragma unroll
            for (int e = 0; e < N; e += 2)
                w[e / 2] = pack2<T>(in[e], in[e + 1]);
        }
        buf_store_words<BYTES / 4, POLICY>(r, off, w);
    }
}

// ---- rows of 2-byte elements ------------------------------------------------------
// Vector accesses go by 32-bit words. A row of 2-byte elements may start at the
// upper half of a word: a crop, a row pitch of an odd number of elements, or a
// detail band whose column offset is odd. All lanes of a row share its
// misalignment, so a load takes the words that hold the lane's elements (one
// more than they fill) and shifts them into place, and a store writes halves
// at its ends and whole words between. Element by element, as before, 4096^2
// one-level FP16 took 23.5 us forward and 23.4 inverse as a crop of an odd
// pitch, and takes 18.2 and 16.4; FP32 crops, whose rows were never off a word
// but off the vector, took 33.2 and 34.0 and take 21.9 and 22.2; 12142 x 14348
// BF16 forward 244 -> 163.
//
// The hardware checks each word of an access against the row's end by itself,
// so a vector may start inside the row and reach past it: a load returns 0
// for the words beyond, a store drops them.

// N elements of T per lane from one row. ODD (2-byte elements): the row may
// start at the upper half of a word.
template <typename T, int N, bool ODD>
struct RowIn {
    static constexpr bool HALF = sizeof(T) == 2 && N > 1;
    static constexpr bool SHIFT = HALF && ODD;
    rsrc_t r;
    uint32_t shift;   // bits; wavefront-uniform

    __device__ __forceinline__ void at(const T *row, int n) {
        uintptr_t a = (uintptr_t)row;
        uint32_t bytes = (uint32_t)n * (uint32_t)sizeof(T);
        if constexpr (SHIFT) {
            shift = (uint32_t)(a & 2u) * 8u;
            bytes += (uint32_t)(a & 2u);
            a &= ~(uintptr_t)3;
        }
        // up to the end of the word that holds the last element
        if constexpr (HALF) bytes = (bytes + 3u) & ~3u;
        r = make_rsrc(reinterpret_cast<const void *>(a), bytes);
    }
    __device__ __forceinline__ void load(uint32_t off, float (&v)[N]) const {
        if constexpr (!SHIFT) {
            load_vec<T, N>(r, off, v);
        } else {
            uint32_t w[N / 2 + 1];
            buf_load_words<N / 2 + 1>(r, off, w);
#pragma unroll
            for (int i = 0; i < N / 2; ++i) {
                const uint32_t x = __builtin_amdgcn_alignbit(w[i + 1], w[i], shift);
                v[2 * i] = Storage<T>::decode(x & 0xffffu);
                v[2 * i + 1] = Storage<T>::decode(x >> 16);
            }
        }
    }
};

// Stores N elements per lane at columns x0.. of a row of n; `on`: the lane
// stores. `words` (2-byte elements; wavefront-uniform): the row is known to
// start at a word. RAGGED: n may be no multiple of N (2-byte elements: the test
// for it makes a basic block of every row; without it 4096^2 one-level FP16 takes
// 16.1 us instead of 16.7 forward, 13.7 instead of 13.9 inverse). Nothing outside
// the row is written.
template <typename T, int N, int POLICY, bool RAGGED>
__device__ __forceinline__ void store_cols(const T *row, int n, int x0, bool on, bool words,
                                           const float (&v)[N]) {
    const uint32_t bytes = (uint32_t)n * (uint32_t)sizeof(T);
    if constexpr (sizeof(T) == 4) {
        store_vec<T, N, POLICY>(make_rsrc(row, bytes), on ? 4u * (uint32_t)x0 : kNoAccess, v);
    } else if constexpr (N == 1) {
        store_elem<T>(make_rsrc(row, bytes), on ? 2u * (uint32_t)x0 : kNoAccess, v[0]);
    } else {
        const uint32_t odd = words ? 0u : (uint32_t)((uintptr_t)row & 2u);
        const rsrc_t r = make_rsrc(reinterpret_cast<const void *>((uintptr_t)row - odd), bytes + odd);
        const uint32_t at = 2u * (uint32_t)x0;
        const uint32_t off = on && (!RAGGED || x0 + N <= n) ? at : kNoAccess;
        if (odd == 0) {   // wavefront-uniform
            store_vec<T, N, POLICY>(r, off, v);
        } else {
            uint32_t w[N / 2];
#pragma unroll
            for (int i = 0; i < N; i += 2) w[i / 2] = pack2<T>(v[i], v[i + 1]);
            __builtin_amdgcn_raw_buffer_store_b16((unsigned short)w[0], r, (int)(off + 2u), 0, POLICY);
#pragma unroll
            for (int i = 1; i < N / 2; ++i)
                __builtin_amdgcn_raw_buffer_store_b32(__builtin_amdgcn_alignbit(w[i], w[i - 1], 16),
                                                      r, (int)(off + 4u * i), 0, POLICY);
            __builtin_amdgcn_raw_buffer_store_b16((unsigned short)(w[N / 2 - 1] >> 16), r,
                                                  (int)(off + 2u * N), 0, POLICY);
        }
        if (RAGGED && on && x0 + N > n) {   // the row's last lane
#pragma unroll
            for (int i = 0; i < N; ++i)
                store_elem<T>(r, x0 + i < n ? at + odd + 2u * i : kNoAccess, v[i]);
        }
    }
}

// ---- boundary ---------------------------------------------------------------
// Whole-sample symmetric extension of an n-sample axis (n >= 2), periodic
// with period 2n-2: the index of the sample that position x stands for.
__device__ __forceinline__ int mirror(int x, int n) {
    if (x < 0) x = -x;                 // the extension is even about 0
    if (x < n) return x;
    const int period = 2 * n - 2;
    if (x >= period) x %= period;      // only for windows wider than the level
    return x < n ? x : period - x;
}

// True when every lane of the wavefront has `c` set: a wavefront-uniform
// branch condition. Loads of the two paths then never share an exec mask,
// so the vector path's loads of all rows stay in flight together.
__device__ __forceinline__ bool wave_all(bool c) {
    return __builtin_amdgcn_ballot_w64(!c) == 0;
}

// ---- cross-lane shifts (DPP, wavefront-wide) ----------------------------------
// from_right(v): lane l receives lane l+1's v (lane 63 receives 0).
// from_left(v):  lane l receives lane l-1's v (lane 0 receives 0).
// The zero for the lane without a source comes from the bound-control bit,
// not from the instruction's old value, so no register has to be zeroed
// before each shift.
__device__ __forceinline__ float from_right(float v) {
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x130, 0xf, 0xf, true));
}
__device__ __forceinline__ float from_left(float v) {
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x138, 0xf, 0xf, true));
}

// ---- the register tile --------------------------------------------------------
template <int ROWS, int QPL>
struct Quads {
    float a[ROWS][QPL], b[ROWS][QPL], c[ROWS][QPL], d[ROWS][QPL];
};

// Mailbox between vertically adjacent wavefronts. Two buffers alternate so
// that one barrier per exchange suffices: the writes of exchange k+1 go to the
// buffer last read in exchange k-1, which every wave finished before it
// passed the barrier of exchange k.
template <int QPL, int WAVES>
struct Mailbox {
    float v[2][WAVES][2][QPL][64];
};

template <int ROWS, int QPL, int WAVES>
struct Exchange {
    Mailbox<QPL, WAVES> *box;
    int wave, lane, buf;

    // Every wave sends its first row's (x, y) up and receives the first row of
    // the wave below it (the row after its last row).
    __device__ __forceinline__ void from_below(const float (&x0)[QPL], const float (&y0)[QPL],
                                               float (&xo)[QPL], float (&yo)[QPL]) {
        if constexpr (WAVES == 1) {
#pragma unroll
            for (int i = 0; i < QPL; ++i) { xo[i] = x0[i]; yo[i] = y0[i]; }
        } else {
#pragma unroll
            for (int i = 0; i < QPL; ++i) {
                box->v[buf][wave][0][i][lane] = x0[i];
                box->v[buf][wave][1][i][lane] = y0[i];
            }
            __syncthreads();
            const int src = (wave + 1 < WAVES) ? wave + 1 : wave;
#pragma unroll
            for (int i = 0; i < QPL; ++i) {
                xo[i] = box->v[buf][src][0][i][lane];
                yo[i] = box->v[buf][src][1][i][lane];
            }
            buf ^= 1;
        }
    }

    // Every wave sends its last row's (x, y) down and receives the last row of
    // the wave above it (the row before its first row).
    __device__ __forceinline__ void from_above(const float (&xl)[QPL], const float (&yl)[QPL],
                                               float (&xo)[QPL], float (&yo)[QPL]) {
        if constexpr (WAVES == 1) {
#pragma unroll
            for (int i = 0; i < QPL; ++i) { xo[i] = xl[i]; yo[i] = yl[i]; }
        } else {
#pragma unroll
            for (int i = 0; i < QPL; ++i) {
                box->v[buf][wave][0][i][lane] = xl[i];
                box->v[buf][wave][1][i][lane] = yl[i];
            }
            __syncthreads();
            const int src = (wave > 0) ? wave - 1 : wave;
#pragma unroll
            for (int i = 0; i < QPL; ++i) {
                xo[i] = box->v[buf][src][0][i][lane];
                yo[i] = box->v[buf][src][1][i][lane];
            }
            buf ^= 1;
        }
    }
};

// ---- non-separable steps (Sec. 3) ---------------------------------------------
// T_P:  b += P a;  c += P* a;  d += P P* a + P* b + P c   (pre-step values)
// S_U:  a += U b + U* c + U U* d;  b += U* d;  c += U d   (pre-step values)
// each as one spatial step with one exchange. The b (low x, high y) term of
// T_P's d and of S_U's a is taken after b's own update, P* (b + P a) being
// P* b + P P* a: the product terms P P*, U U* then cost nothing (8 operations
// per quad and step, against 9 with them written out). Every two-tap filter
// adds its two neighbours first and multiplies once. Addition commutes, so a
// step gives the same bits on mirrored data: a symmetrically extended signal
// stays symmetric to the last bit, and a kernel may either carry the extension
// along as halo quads or put a quad's own value in a missing neighbour's
// place (p (x + x) at the right and lower edge, u (y + y) at the left and
// upper) and get the same result. Against 64 bits, relative 2-norm, one level
// of 1024^2 in FP32 (with one FMA per tap): 9/7 forward 3.7e-7 (4.7e-7), inverse
// 3.0e-7 (3.5e-7); 5/3 inverse of a smooth picture 4.3e-8 (4.9e-8), but its
// forward 6.2e-8 (5.6e-8): there the sum of two neighbours rounds at the pixels'
// magnitude, not at the detail's. 8-bit pictures are exact in 5/3. T_P's d takes
// the c pair and the b pair one after the other (one sum of four: 9/7 3.8e-7,
// 5/3 7.1e-8), S_U's a takes one sum (two: 3.8e-7, 6.7e-8).
template <int QPL>
__device__ __forceinline__ void add_right(const float (&x)[QPL], float (&s)[QPL]) {
    const float xr = from_right(x[0]);
#pragma unroll
    for (int i = 0; i < QPL; ++i) s[i] = x[i] + ((i + 1 < QPL) ? x[(i + 1 < QPL) ? i + 1 : i] : xr);
}
template <int QPL>
__device__ __forceinline__ void add_left(const float (&x)[QPL], float (&s)[QPL]) {
    const float xl = from_left(x[QPL - 1]);
#pragma unroll
    for (int i = 0; i < QPL; ++i) s[i] = x[i] + ((i > 0) ? x[(i > 0) ? i - 1 : i] : xl);
}

template <int ROWS, int QPL, int WAVES>
__device__ __forceinline__ void nonsep_predict(Quads<ROWS, QPL> &q, Exchange<ROWS, QPL, WAVES> &x,
                                               float p) {
#pragma unroll
    for (int r = 0; r < ROWS; ++r) {   // b: horizontal, own row only
        float s[QPL];
        add_right(q.a[r], s);
#pragma unroll
        for (int i = 0; i < QPL; ++i) q.b[r][i] = fmaf(p, s[i], q.b[r][i]);
    }
    float na[QPL], nb[QPL];
    x.from_below(q.a[0], q.b[0], na, nb);
#pragma unroll
    for (int r = 0; r < ROWS; ++r) {
        float s[QPL];
        add_right(q.c[r], s);
#pragma unroll
        for (int i = 0; i < QPL; ++i) {
            const float ad = (r + 1 < ROWS) ? q.a[(r + 1 < ROWS) ? r + 1 : r][i] : na[i];
            const float bd = (r + 1 < ROWS) ? q.b[(r + 1 < ROWS) ? r + 1 : r][i] : nb[i];
            q.d[r][i] = fmaf(p, q.b[r][i] + bd, fmaf(p, s[i], q.d[r][i]));
            q.c[r][i] = fmaf(p, q.a[r][i] + ad, q.c[r][i]);
        }
    }
}

// Rows run bottom to top so that the row above still holds its pre-step c.
template <int ROWS, int QPL, int WAVES>
__device__ __forceinline__ void nonsep_update(Quads<ROWS, QPL> &q, Exchange<ROWS, QPL, WAVES> &x,
                                              float u) {
    float pc[QPL], pd[QPL];
    x.from_above(q.c[ROWS - 1], q.d[ROWS - 1], pc, pd);
#pragma unroll
    for (int r = ROWS - 1; r >= 0; --r) {
        float sd[QPL], sb[QPL];
        add_left(q.d[r], sd);
#pragma unroll
        for (int i = 0; i < QPL; ++i) {
            const float du = (r > 0) ? q.d[(r > 0) ? r - 1 : r][i] : pd[i];
            q.b[r][i] = fmaf(u, q.d[r][i] + du, q.b[r][i]);
        }
        add_left(q.b[r], sb);
#pragma unroll
        for (int i = 0; i < QPL; ++i) {
            const float cu = (r > 0) ? q.c[(r > 0) ? r - 1 : r][i] : pc[i];
            q.a[r][i] = fmaf(u, sb[i] + (q.c[r][i] + cu), q.a[r][i]);
            q.c[r][i] = fmaf(u, sd[i], q.c[r][i]);
        }
    }
}

// ---- separable steps (Sec. 2) -------------------------------------------------
// T^H_P: b += P a, d += P c.  Horizontal only: DPP exchange, no barrier.
template <int ROWS, int QPL>
__device__ __forceinline__ void sep_predict_h(Quads<ROWS, QPL> &q, float p) {
#pragma unroll
    for (int r = 0; r < ROWS; ++r) {
        float sa[QPL], sc[QPL];
        add_right(q.a[r], sa);
        add_right(q.c[r], sc);
#pragma unroll
        for (int i = 0; i < QPL; ++i) {
            q.b[r][i] = fmaf(p, sa[i], q.b[r][i]);
            q.d[r][i] = fmaf(p, sc[i], q.d[r][i]);
        }
    }
}

// T^V_P: c += P* a, d += P* b.  Vertical: one mailbox exchange.
template <int ROWS, int QPL, int WAVES>
__device__ __forceinline__ void sep_predict_v(Quads<ROWS, QPL> &q, Exchange<ROWS, QPL, WAVES> &x,
                                              float p) {
    float na[QPL], nb[QPL];
    x.from_below(q.a[0], q.b[0], na, nb);
#pragma unroll
    for (int r = 0; r < ROWS; ++r) {
#pragma unroll
        for (int i = 0; i < QPL; ++i) {
            const float ad = (r + 1 < ROWS) ? q.a[(r + 1 < ROWS) ? r + 1 : r][i] : na[i];
            const float bd = (r + 1 < ROWS) ? q.b[(r + 1 < ROWS) ? r + 1 : r][i] : nb[i];
            q.c[r][i] = fmaf(p, q.a[r][i] + ad, q.c[r][i]);
            q.d[r][i] = fmaf(p, q.b[r][i] + bd, q.d[r][i]);
        }
    }
}

// S^H_U: a += U b, c += U d.
template <int ROWS, int QPL>
__device__ __forceinline__ void sep_update_h(Quads<ROWS, QPL> &q, float u) {
#pragma unroll
    for (int r = 0; r < ROWS; ++r) {
        float sb[QPL], sd[QPL];
        add_left(q.b[r], sb);
        add_left(q.d[r], sd);
#pragma unroll
        for (int i = 0; i < QPL; ++i) {
            q.a[r][i] = fmaf(u, sb[i], q.a[r][i]);
            q.c[r][i] = fmaf(u, sd[i], q.c[r][i]);
        }
    }
}

// S^V_U: a += U* c, b += U* d.
template <int ROWS, int QPL, int WAVES>
__device__ __forceinline__ void sep_update_v(Quads<ROWS, QPL> &q, Exchange<ROWS, QPL, WAVES> &x,
                                             float u) {
    float pc[QPL], pd[QPL];
    x.from_above(q.c[ROWS - 1], q.d[ROWS - 1], pc, pd);
#pragma unroll
    for (int r = 0; r < ROWS; ++r) {
#pragma unroll
        for (int i = 0; i < QPL; ++i) {
            const float cu = (r > 0) ? q.c[(r > 0) ? r - 1 : r][i] : pc[i];
            const float du = (r > 0) ? q.d[(r > 0) ? r - 1 : r][i] : pd[i];
            q.a[r][i] = fmaf(u, q.c[r][i] + cu, q.a[r][i]);
            q.b[r][i] = fmaf(u, q.d[r][i] + du, q.b[r][i]);
        }
    }
}

// ---- every exchange through LDS (ablation of the DPP lane shifts) ------------
// Per-row edge values of each lane, double-buffered like the mailbox; one
// exchange publishes, passes one workgroup barrier and reads.
template <int ROWS, int WAVES>
struct HBox {
    float v[2][WAVES][2][ROWS][64];
};

template <int ROWS, int QPL, int WAVES>
struct LdsExchange {
    Mailbox<QPL, WAVES> *box;
    HBox<ROWS, WAVES> *hb;
    int wave, lane, buf;
};

// T_P with the right neighbours (a, c of the next lane's first quad, and the
// row below) and the lower row read from LDS after one barrier.
template <int ROWS, int QPL, int WAVES>
__device__ __forceinline__ void nonsep_predict_lds(Quads<ROWS, QPL> &q,
                                                   LdsExchange<ROWS, QPL, WAVES> &x, float p) {
    const int b = x.buf, w = x.wave, l = x.lane;
#pragma unroll
    for (int r = 0; r < ROWS; ++r) {
        x.hb->v[b][w][0][r][l] = q.a[r][0];
        x.hb->v[b][w][1][r][l] = q.c[r][0];
    }
#pragma unroll
    for (int i = 0; i < QPL; ++i) {
        x.box->v[b][w][0][i][l] = q.a[0][i];
        x.box->v[b][w][1][i][l] = q.b[0][i];
    }
    __syncthreads();
    const int src = (w + 1 < WAVES) ? w + 1 : w;
    const int rl = l < 63 ? l + 1 : l;      // the window's last lane reads itself
    float na[QPL], nb[QPL];
#pragma unroll
    for (int i = 0; i < QPL; ++i) {
        na[i] = x.box->v[b][src][0][i][l];
        nb[i] = x.box->v[b][src][1][i][l];
    }
    float aR[ROWS], cR[ROWS];
#pragma unroll
    for (int r = 0; r < ROWS; ++r) {
        aR[r] = x.hb->v[b][w][0][r][rl];
        cR[r] = x.hb->v[b][w][1][r][rl];
    }
    const float naR = x.box->v[b][src][0][0][rl];
    x.buf ^= 1;
#pragma unroll
    for (int i = 0; i < QPL; ++i) {   // b of every row, and of the row below the last
#pragma unroll
        for (int r = 0; r < ROWS; ++r) {
            const float ar = (i + 1 < QPL) ? q.a[r][(i + 1 < QPL) ? i + 1 : i] : aR[r];
            q.b[r][i] = fmaf(p, q.a[r][i] + ar, q.b[r][i]);
        }
        nb[i] = fmaf(p, na[i] + ((i + 1 < QPL) ? na[(i + 1 < QPL) ? i + 1 : i] : naR), nb[i]);
    }
#pragma unroll
    for (int r = 0; r < ROWS; ++r) {
#pragma unroll
        for (int i = 0; i < QPL; ++i) {
            const float ad = (r + 1 < ROWS) ? q.a[(r + 1 < ROWS) ? r + 1 : r][i] : na[i];
            const float bd = (r + 1 < ROWS) ? q.b[(r + 1 < ROWS) ? r + 1 : r][i] : nb[i];
            const float c = q.c[r][i];
            const float cr = (i + 1 < QPL) ? q.c[r][(i + 1 < QPL) ? i + 1 : i] : cR[r];
            q.d[r][i] = fmaf(p, q.b[r][i] + bd, fmaf(p, c + cr, q.d[r][i]));
            q.c[r][i] = fmaf(p, q.a[r][i] + ad, c);
        }
    }
}

// S_U with the left neighbours (b, d of the previous lane's last quad, and the
// row above) and the upper row read from LDS after one barrier.
template <int ROWS, int QPL, int WAVES>
__device__ __forceinline__ void nonsep_update_lds(Quads<ROWS, QPL> &q,
                                                  LdsExchange<ROWS, QPL, WAVES> &x, float u) {
    const int b = x.buf, w = x.wave, l = x.lane;
#pragma unroll
    for (int r = 0; r < ROWS; ++r) {
        x.hb->v[b][w][0][r][l] = q.b[r][QPL - 1];
        x.hb->v[b][w][1][r][l] = q.d[r][QPL - 1];
    }
#pragma unroll
    for (int i = 0; i < QPL; ++i) {
        x.box->v[b][w][0][i][l] = q.c[ROWS - 1][i];
        x.box->v[b][w][1][i][l] = q.d[ROWS - 1][i];
    }
    __syncthreads();
    const int src = (w > 0) ? w - 1 : w;
    const int ll = l > 0 ? l - 1 : l;       // the window's first lane reads itself
    float pc[QPL], pd[QPL];
#pragma unroll
    for (int i = 0; i < QPL; ++i) {
        pc[i] = x.box->v[b][src][0][i][l];
        pd[i] = x.box->v[b][src][1][i][l];
    }
    float bL[ROWS], dL[ROWS], duL[ROWS];
#pragma unroll
    for (int r = 0; r < ROWS; ++r) {
        bL[r] = x.hb->v[b][w][0][r][ll];
        dL[r] = x.hb->v[b][w][1][r][ll];
        duL[r] = (r > 0) ? x.hb->v[b][w][1][(r > 0) ? r - 1 : r][ll]
                         : x.box->v[b][src][1][QPL - 1][ll];
    }
    x.buf ^= 1;
#pragma unroll
    for (int r = ROWS - 1; r >= 0; --r) {
        // the left lane's b after its update, as that lane computes it
        float bl = fmaf(u, dL[r] + duL[r], bL[r]);
        float dl = dL[r];
#pragma unroll
        for (int i = 0; i < QPL; ++i) {
            const float cu = (r > 0) ? q.c[(r > 0) ? r - 1 : r][i] : pc[i];
            const float du = (r > 0) ? q.d[(r > 0) ? r - 1 : r][i] : pd[i];
            const float c = q.c[r][i], d = q.d[r][i];
            const float bv = fmaf(u, d + du, q.b[r][i]);
            q.a[r][i] = fmaf(u, (bv + bl) + (c + cu), q.a[r][i]);
            q.c[r][i] = fmaf(u, d + dl, c);
            q.b[r][i] = bv;
            bl = bv;
            dl = d;
        }
    }
}

// T^H_P through LDS: one barrier.
template <int ROWS, int QPL, int WAVES>
__device__ __forceinline__ void sep_predict_h_lds(Quads<ROWS, QPL> &q,
                                                  LdsExchange<ROWS, QPL, WAVES> &x, float p) {
    const int b = x.buf, w = x.wave, l = x.lane;
#pragma unroll
    for (int r = 0; r < ROWS; ++r) {
        x.hb->v[b][w][0][r][l] = q.a[r][0];
        x.hb->v[b][w][1][r][l] = q.c[r][0];
    }
    __syncthreads();
    const int rl = l < 63 ? l + 1 : l;
    float aR[ROWS], cR[ROWS];
#pragma unroll
    for (int r = 0; r < ROWS; ++r) {
        aR[r] = x.hb->v[b][w][0][r][rl];
        cR[r] = x.hb->v[b][w][1][r][rl];
    }
    x.buf ^= 1;
#pragma unroll
    for (int r = 0; r < ROWS; ++r) {
#pragma unroll
        for (int i = 0; i < QPL; ++i) {
            const float ar = (i + 1 < QPL) ? q.a[r][(i + 1 < QPL) ? i + 1 : i] : aR[r];
            const float cr = (i + 1 < QPL) ? q.c[r][(i + 1 < QPL) ? i + 1 : i] : cR[r];
            q.b[r][i] = fmaf(p, q.a[r][i] + ar, q.b[r][i]);
            q.d[r][i] = fmaf(p, q.c[r][i] + cr, q.d[r][i]);
        }
    }
}

// S^H_U through LDS: one barrier.
template <int ROWS, int QPL, int WAVES>
__device__ __forceinline__ void sep_update_h_lds(Quads<ROWS, QPL> &q,
                                                 LdsExchange<ROWS, QPL, WAVES> &x, float u) {
    const int b = x.buf, w = x.wave, l = x.lane;
#pragma unroll
    for (int r = 0; r < ROWS; ++r) {
        x.hb->v[b][w][0][r][l] = q.b[r][QPL - 1];
        x.hb->v[b][w][1][r][l] = q.d[r][QPL - 1];
    }
    __syncthreads();
    const int ll = l > 0 ? l - 1 : l;
    float bL[ROWS], dL[ROWS];
#pragma unroll
    for (int r = 0; r < ROWS; ++r) {
        bL[r] = x.hb->v[b][w][0][r][ll];
        dL[r] = x.hb->v[b][w][1][r][ll];
    }
    x.buf ^= 1;
#pragma unroll
    for (int r = 0; r < ROWS; ++r) {
#pragma unroll
        for (int i = 0; i < QPL; ++i) {
            const float bl = (i > 0) ? q.b[r][(i > 0) ? i - 1 : i] : bL[r];
            const float dl = (i > 0) ? q.d[r][(i > 0) ? i - 1 : i] : dL[r];
            q.a[r][i] = fmaf(u, q.b[r][i] + bl, q.a[r][i]);
            q.c[r][i] = fmaf(u, q.d[r][i] + dl, q.c[r][i]);
        }
    }
}

// The vertical separable steps on the LDS exchange's mailbox (same parity).
template <int ROWS, int QPL, int WAVES>
__device__ __forceinline__ Exchange<ROWS, QPL, WAVES> as_exchange(LdsExchange<ROWS, QPL, WAVES> &x) {
    return Exchange<ROWS, QPL, WAVES>{x.box, x.wave, x.lane, x.buf};
}

// ---- whole lifting sequences --------------------------------------------------
template <int WV, int SCH, int ROWS, int QPL, int WAVES>
__device__ __forceinline__ void lift_forward(Quads<ROWS, QPL> &q, LdsExchange<ROWS, QPL, WAVES> &x) {
    using L = Wavelet<WV>;
#pragma unroll
    for (int k = 0; k < L::NPAIRS; ++k) {
        const float p = (float)L::p(k), u = (float)L::u(k);
        if constexpr (SCH == NONSEP_LDS) {
            nonsep_predict_lds(q, x, p);
            nonsep_update_lds(q, x, u);
        } else {
            sep_predict_h_lds(q, x, p);
            Exchange<ROWS, QPL, WAVES> v = as_exchange(x);
            sep_predict_v(q, v, p);
            x.buf = v.buf;
            sep_update_h_lds(q, x, u);
            v = as_exchange(x);
            sep_update_v(q, v, u);
            x.buf = v.buf;
        }
    }
}

template <int WV, int SCH, int ROWS, int QPL, int WAVES>
__device__ __forceinline__ void lift_inverse(Quads<ROWS, QPL> &q, LdsExchange<ROWS, QPL, WAVES> &x) {
    using L = Wavelet<WV>;
#pragma unroll
    for (int k = L::NPAIRS - 1; k >= 0; --k) {
        const float p = -(float)L::p(k), u = -(float)L::u(k);
        if constexpr (SCH == NONSEP_LDS) {
            nonsep_update_lds(q, x, u);
            nonsep_predict_lds(q, x, p);
        } else {
            Exchange<ROWS, QPL, WAVES> v = as_exchange(x);
            sep_update_v(q, v, u);
            x.buf = v.buf;
            sep_update_h_lds(q, x, u);
            v = as_exchange(x);
            sep_predict_v(q, v, p);
            x.buf = v.buf;
            sep_predict_h_lds(q, x, p);
        }
    }
}

template <int WV, int SCH, int ROWS, int QPL, int WAVES>
__device__ __forceinline__ void lift_forward(Quads<ROWS, QPL> &q, Exchange<ROWS, QPL, WAVES> &x) {
    using L = Wavelet<WV>;
#pragma unroll
    for (int k = 0; k < L::NPAIRS; ++k) {
        const float p = (float)L::p(k), u = (float)L::u(k);
        if constexpr (SCH == NONSEP) {
            nonsep_predict(q, x, p);
            nonsep_update(q, x, u);
        } else {
            sep_predict_h(q, p);
            sep_predict_v(q, x, p);
            sep_update_h(q, u);
            sep_update_v(q, x, u);
        }
    }
}

// The inverse undoes each step with the negated filter, in reverse order.
template <int WV, int SCH, int ROWS, int QPL, int WAVES>
__device__ __forceinline__ void lift_inverse(Quads<ROWS, QPL> &q, Exchange<ROWS, QPL, WAVES> &x) {
    using L = Wavelet<WV>;
#pragma unroll
    for (int k = L::NPAIRS - 1; k >= 0; --k) {
        const float p = -(float)L::p(k), u = -(float)L::u(k);
        if constexpr (SCH == NONSEP) {
            nonsep_update(q, x, u);
            nonsep_predict(q, x, p);
        } else {
            sep_update_v(q, x, u);
            sep_update_h(q, u);
            sep_predict_v(q, x, p);
            sep_predict_h(q, p);
        }
    }
}

}  // namespace dwt2
