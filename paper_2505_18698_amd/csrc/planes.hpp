// fp32 products on the bf16 matrix instruction.  An fp32 value is the sum of
// three bf16 values (its planes: the leading 8 bits, the next 8, the rest), an
// fp16 value of two, a bf16 value of one.  A product runs on the 16x16x32
// instruction (16 times the rate of the fp32 16x16x4 one) once for every pair
// of planes p, q with p + q <= 2, accumulating in fp32.  The pairs left out
// are at most 2^-24 of it, the rounding of one fp32 multiply, and below 2^-26
// for 97% of uniform operands.
//
// Range.  The sum is exact for finite values from 2^-110 up.  The instruction
// takes bf16 values below 2^-126 as zero, so a smaller operand keeps 16 bits
// (from 2^-117 up) or 8: a gradient that is 2^-115 as a whole has a relative
// error of 3e-3, one of 2^-100 that of any other.  Sums of products may round to
// an infinity where they come within 2^-16 of the end of fp32's range.  An
// infinity is not a sum of planes; Reach::kInf says what stands for it.
#pragma once

#include "tiles.hpp"

namespace ma {

typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));

// bf16 planes of an element type (split).
template <typename T> constexpr int planes_of = std::is_same<T, float>::value ? 3 : std::is_same<T, __bf16>::value ? 1 : 2;

// Which values the planes of an operand stand for.
enum class Reach {
    kUnit,    // factors of a softmax: nothing near the end of fp32's range
    kFinite,  // every finite value: one more instruction an element, as those beyond
              // 3.396e38 would round to an infinite leading plane; an infinity gives NaN
    kInf,     // infinities too.  In three planes an infinity is a finite leading plane, a
              // finite second one, and itself: the last plane meets only the other
              // operand's leading plane, which is zero exactly where the operand is, so
              // its products with a factor are infinite, or NaN with a zero, as those of
              // the fp32 instruction.  In two planes itself and a finite value
              // (mma_planes_inf).
};

// x[0..N) as the sum of NP bf16 planes, each the nearest bf16 value of what
// the planes before it leave.  (The median of NaN and two bounds is one of
// them: a NaN is kept by the last plane.)
template <int NP, int N, Reach R, typename V> __device__ inline void split(const float *x, V (&p)[NP])
{
    float r[N];
#pragma unroll
    for (int i = 0; i < N; ++i) r[i] = x[i];
#pragma unroll
    for (int a = 0; a < NP; ++a) {
        // bounds of plane a: the largest bf16 value, or more than a lower plane of a finite value reaches
        constexpr float kTop = 3.38953139e38f, kRest = NP == 3 ? 0x1p121f : 256.f;
        const bool bound = NP == 3 ? (a == 0 && R != Reach::kUnit) || (a == 1 && R == Reach::kInf) : (a == 1 && R == Reach::kInf);
        const float lim = a == 0 ? kTop : kRest;
#pragma unroll
        for (int i = 0; i < N; i += 2) {  // two at a time: one conversion, and the halves of its result back as floats
            const float y0 = bound ? __builtin_amdgcn_fmed3f(r[i], -lim, lim) : r[i];
            const float y1 = bound ? __builtin_amdgcn_fmed3f(r[i + 1], -lim, lim) : r[i + 1];
            const bf16x2 h = __builtin_convertvector((f32x2{y0, y1}), bf16x2);
            p[a][i] = h[0];
            p[a][i + 1] = h[1];
            if (a + 1 < NP) {
                uint32_t u;
                __builtin_memcpy(&u, &h, 4);
                r[i] -= __uint_as_float(u << 16);
                r[i + 1] -= __uint_as_float(u & 0xffff0000u);
            }
        }
    }
}

__device__ inline f32x4 mfma(bf16x8 a, bf16x8 b, f32x4 c) { return Mma<__bf16>::mma(a, b, c); }
__device__ inline f32x4 mfma(bf16x4 a, bf16x4 b, f32x4 c) { return Mma<__bf16>::mma4(a, b, c); }

// c += sum over the plane pairs, the smallest first.
template <int NA, int NB, typename F> __device__ inline void mma_planes(const F (&a)[NA], const F (&b)[NB], f32x4 &c)
{
#pragma unroll
    for (int s = 2; s >= 0; --s) {
#pragma unroll
        for (int i = 0; i < NA; ++i) {
            const int j = s - i;
            if (j >= 0 && j < NB) c = mfma(a[i], b[j], c);
        }
    }
}

// A plane with its infinities (and NaN) replaced by the largest finite value.
template <typename F> __device__ inline F finite_plane(F x)
{
    typedef unsigned short words __attribute__((ext_vector_type(sizeof(F) / 2)));
    words w;
    __builtin_memcpy(&w, &x, sizeof(F));
    const words top = (words)(unsigned short)0x7f7f, sign = (words)(unsigned short)0x8000;
    w = __builtin_elementwise_min(w & ~sign, top) | (w & sign);
    __builtin_memcpy(&x, &w, sizeof(F));
    return x;
}

// mma_planes where a, of Reach::kInf, may hold infinities and b is a factor: in
// one or two planes they meet b's leading plane only (its others can be zero,
// or negative).
template <int NA, typename F> __device__ inline void mma_planes_inf(const F (&a)[NA], const F (&b)[3], f32x4 &c)
{
    if constexpr (NA == 3) {
        mma_planes(a, b, c);
    } else {
        const F fin = finite_plane(a[0]);
        c = mfma(fin, b[2], c);
        if constexpr (NA == 2) c = mfma(a[1], b[1], c);
        c = mfma(fin, b[1], c);
        if constexpr (NA == 2) c = mfma(a[1], b[0], c);
        c = mfma(a[0], b[0], c);
        if constexpr (NA == 2) __builtin_amdgcn_sched_barrier(0);  // one tile's planes at a time (fewer spills at 128 x 128)
    }
}

// The scores and the factor's gradient, which the softmax and its pull-back
// amplify: fp32 elements sum the leading planes' product (hi) apart from the
// five small ones (lo), so that it takes one rounding a chunk and not six.
template <bool TWO> struct Score {
    f32x4 hi, lo;
    __device__ Score() : hi{0.f, 0.f, 0.f, 0.f}, lo{0.f, 0.f, 0.f, 0.f} {}
    template <int NA, int NB> __device__ inline void add(const bf16x8 (&a)[NA], const bf16x8 (&b)[NB])
    {
        if constexpr (TWO) {
            hi = mfma(a[0], b[0], hi);
#pragma unroll
            for (int s = 2; s >= 1; --s) {
#pragma unroll
                for (int i = 0; i < NA; ++i) {
                    const int j = s - i;
                    if (j >= 0 && j < NB) lo = mfma(a[i], b[j], lo);
                }
            }
        } else {
            mma_planes(a, b, hi);
        }
    }
    __device__ inline f32x4 value() const { return TWO ? hi + lo : hi; }
};

// Operand fragments of the products that contract over KD = 32 or 16 rows or
// columns of a unit (KD = 16 only where the unit has no more).
template <int KD> using Frag = typename std::conditional<KD == 32, bf16x8, bf16x4>::type;

// Rows x0 .. x0 + KD - 1 (the contraction index), column c0 + lane % 16, of
// every plane of a row-major LDS tile: slots 0..3 of lane group g are rows
// 4g + q, slots 4..7 rows 16 + 4g + q.
template <int KD, int NP>
__device__ inline void read_cols(const __bf16 *X, int plane, int ld, int x0, int c0, int lane, Frag<KD> (&f)[NP])
{
#pragma unroll
    for (int a = 0; a < NP; ++a) {
        const bf16x4 lo = rows4<__bf16>(X + a * plane, ld, x0, c0, lane);
        if constexpr (KD == 32) {
            const bf16x4 hi = rows4<__bf16>(X + a * plane, ld, x0 + 16, c0, lane);
            f[a] = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
        } else {
            f[a] = lo;
        }
    }
}

// Columns c0 .. c0 + KD - 1 (the contraction index) of row `row` of every
// plane, in the slots of read_cols.
template <int KD, int NP>
__device__ inline void read_row(const __bf16 *row, int plane, int c0, int g, Frag<KD> (&f)[NP])
{
#pragma unroll
    for (int a = 0; a < NP; ++a) {
        const __bf16 *src = row + a * plane + c0 + 4 * g;
        const bf16x4 lo = *reinterpret_cast<const bf16x4 *>(src);
        if constexpr (KD == 32) {
            const bf16x4 hi = *reinterpret_cast<const bf16x4 *>(src + 16);
            f[a] = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
        } else {
            f[a] = lo;
        }
    }
}

// Elements 32c + 8g .. + 7 of a row of every plane of an LDS tile (products
// that contract over the head dimension).
template <int NP> __device__ inline void read_chunk(const __bf16 *row, int plane, int c, int g, bf16x8 (&f)[NP])
{
#pragma unroll
    for (int a = 0; a < NP; ++a) f[a] = *reinterpret_cast<const bf16x8 *>(row + a * plane + 32 * c + 8 * g);
}

// read_chunk from row `row` of E, d elements apart, in global memory (!ok: zero),
// elements >= d zero (d a multiple of 16 bytes' worth).
template <typename E, int NP> __device__ inline void load_chunk(const Span &s, int row, bool ok, int c, int g, int d, bf16x8 (&f)[NP])
{
    constexpr int V = 16 / (int)sizeof(E);
    E e[8];
#pragma unroll
    for (int v = 0; v < 8; v += V) {
        const int col = 32 * c + 8 * g + v;
        const u32x4 raw = s.load16((row * d + col) * (uint32_t)sizeof(E), ok && col < d);
        __builtin_memcpy(e + v, &raw, 16);
    }
    if constexpr (NP == 1) {
        __builtin_memcpy(&f[0], e, 16);
    } else {
        float x[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) x[i] = static_cast<float>(e[i]);
        split<NP, 8, Reach::kFinite>(x, f);
    }
}

// R rows of D elements of E from global memory into registers (fetch), and
// from there into the NP planes of an LDS tile of row stride LD (stage), the
// 16-byte chunks shared out over NTH threads.  Rows >= nr and columns >= nc
// (a multiple of a chunk) are zero.
template <typename E, int NP, int R, int D, int LD, int NTH, Reach RC = Reach::kFinite> struct Rows {
    static constexpr int V = 16 / (int)sizeof(E), CPR = D / V, ALL = R * CPR, CH = (ALL + NTH - 1) / NTH;
    static constexpr int PLANE = R * LD;
    u32x4 c[CH];

    // Row r is o0 + r * step elements from base (offsets in 32 bits, within a head and not negative).
    __device__ inline void fetch(const E *base, int step, int nr, int nc, int tid, int o0 = 0)
    {
        const Span s(base);
#pragma unroll
        for (int h = 0; h < CH; ++h) {
            const int idx = tid + h * NTH, r = idx / CPR, col = (idx % CPR) * V;
            c[h] = s.load16((uint32_t)(o0 + r * step + col) * (uint32_t)sizeof(E), r < nr && col < nc);  // nr <= R
        }
    }

    __device__ inline void stage(__bf16 *X, int tid) const
    {
#pragma unroll
        for (int h = 0; h < CH; ++h) {
            const int idx = tid + h * NTH, r = idx / CPR, col = (idx % CPR) * V;
            if (ALL % NTH != 0 && idx >= ALL) break;
            __bf16 *dst = X + r * LD + col;
            if constexpr (NP == 1) {
                *reinterpret_cast<u32x4 *>(dst) = c[h];
            } else {
                typedef __bf16 vec __attribute__((ext_vector_type(V)));
                E e[V];
                __builtin_memcpy(e, &c[h], 16);
                float x[V];
#pragma unroll
                for (int i = 0; i < V; ++i) x[i] = static_cast<float>(e[i]);
                vec p[NP];
                split<NP, V, RC>(x, p);
#pragma unroll
                for (int a = 0; a < NP; ++a) *reinterpret_cast<vec *>(dst + a * PLANE) = p[a];
            }
        }
    }
};

}  // namespace ma
