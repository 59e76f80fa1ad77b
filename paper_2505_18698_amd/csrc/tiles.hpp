// What the kernels are built from: element types and the matrix instructions,
// cross-lane steps, tiles and operand fragments, and the tensors, states and
// dimensions of a call.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>
#include <type_traits>

namespace ma {

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef _Float16 f16x4 __attribute__((ext_vector_type(4)));
typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef s16x4 __attribute__((address_space(3))) lds_s16x4;

constexpr float kLog2e = 1.4426950408889634f;
constexpr float kLn2 = 0.6931471805599453f;
constexpr float kMasked = -1.0e30f;  // finite "minus infinity": exp2 gives 0 and 0 * kMasked stays 0
constexpr float kTiny = 1.17549435e-38f;

template <typename T> struct Mma;

template <> struct Mma<float> {
    static constexpr int KC = 4;   // contraction length of one instruction
    static constexpr int KPL = 1;  // contraction elements per lane
    using frag = float;
    __device__ static f32x4 mma(frag a, frag b, f32x4 c)
    {
        return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
    }
};

template <> struct Mma<__bf16> {
    static constexpr int KC = 32;
    static constexpr int KPL = 8;
    using frag = bf16x8;
    using frag4 = bf16x4;
    __device__ static f32x4 mma(frag a, frag b, f32x4 c)
    {
        return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
    }
    __device__ static f32x4 mma4(frag4 a, frag4 b, f32x4 c)
    {
        return __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(a, b, c, 0, 0, 0);
    }
};

template <> struct Mma<_Float16> {
    static constexpr int KC = 32;
    static constexpr int KPL = 8;
    using frag = f16x8;
    using frag4 = f16x4;
    __device__ static f32x4 mma(frag a, frag b, f32x4 c)
    {
        return __builtin_amdgcn_mfma_f32_16x16x32_f16(a, b, c, 0, 0, 0);
    }
    __device__ static f32x4 mma4(frag4 a, frag4 b, f32x4 c)
    {
        return __builtin_amdgcn_mfma_f32_16x16x16f16(a, b, c, 0, 0, 0);
    }
};

// Row stride (elements) of a row-major LDS tile with C columns: pad by
// MA_LDS_PAD bytes (32 measured fastest of 0, 16 and 32 on the half-steps).
#ifndef MA_LDS_PAD
#define MA_LDS_PAD 32
#endif
template <typename T, int C> struct Ld {
    static constexpr int row = C + MA_LDS_PAD / (int)sizeof(T);
};

// gfx950's v_permlane16_swap / v_permlane32_swap applied to (x, x) return
// x[lane] and x[lane ^ 16] (resp. x[lane ^ 32]), in an order that depends on
// the lane: a VALU exchange with no LDS round trip.  The pair feeds
// commutative operations only, except in xor16_value.
template <int MASK> __device__ inline void xor_pair(uint32_t x, uint32_t &a, uint32_t &b)
{
    static_assert(MASK == 16 || MASK == 32, "lane distance 16 or 32");
    if constexpr (MASK == 16) {
        const auto r = __builtin_amdgcn_permlane16_swap(x, x, false, false);
        a = r[0];
        b = r[1];
    } else {
        const auto r = __builtin_amdgcn_permlane32_swap(x, x, false, false);
        a = r[0];
        b = r[1];
    }
}

// max(a, b) that propagates NaN (IEEE 754-2019 maximum): one v_maximum3_f32
// on gfx950, where fmaxf first canonicalises each operand with a v_max_f32
// of its own.  The scores are finite or NaN from arithmetic, so the two agree
// wherever neither is NaN, and a NaN reaches the row's maximum either way.
__device__ inline float max_nan(float a, float b) { return __builtin_elementwise_maximum(a, b); }

template <int MASK> __device__ inline float wave_xor_max(float x)
{
    uint32_t a, b;
    xor_pair<MASK>(__float_as_uint(x), a, b);
    return max_nan(__uint_as_float(a), __uint_as_float(b));
}

template <int MASK> __device__ inline float wave_xor_sum(float x)
{
    uint32_t a, b;
    xor_pair<MASK>(__float_as_uint(x), a, b);
    return __uint_as_float(a) + __uint_as_float(b);
}

// x[lane ^ 16]; odd_row = bit 4 of the lane.  The first result of
// permlane16_swap holds the partner in odd rows of 16 lanes, the second in
// even rows.
__device__ inline uint32_t xor16_value(uint32_t x, bool odd_row)
{
    uint32_t a, b;
    xor_pair<16>(x, a, b);
    return odd_row ? a : b;
}

template <typename T> __device__ inline T to_elem(float x) { return static_cast<T>(x); }

// Store 4 consecutive output elements.
template <typename T> __device__ inline void store4(T *dst, f32x4 v)
{
    if constexpr (std::is_same<T, float>::value) {
        *reinterpret_cast<f32x4 *>(dst) = v;
    } else {
        T e[4] = {to_elem<T>(v[0]), to_elem<T>(v[1]), to_elem<T>(v[2]), to_elem<T>(v[3])};
        u32x2 raw;
        __builtin_memcpy(&raw, e, 8);
        *reinterpret_cast<u32x2 *>(dst) = raw;
    }
}

// A uniform base address with 32-bit byte offsets.  A lane whose `ok` is false
// takes an offset past the end: its load gives zero and its store is dropped,
// by the hardware's range check.  No access sits under a branch, so the
// compiler knows how many are in flight: a wait for the rows fetched a chunk
// ago does not also wait for the stores issued since.
struct Span {
    __amdgpu_buffer_rsrc_t r;
    static constexpr int kEnd = 0x7fffffff, kDefault = 0x00027000;  // raw, 32-bit data format
    __device__ explicit Span(const void *base) : r(__builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(base), 0, kEnd, kDefault)) {}
    __device__ static inline int at(uint32_t bytes, bool ok) { return ok ? (int)bytes : (int)0x80000000u; }
    __device__ inline u32x4 load16(uint32_t bytes, bool ok) const
    {
        return __builtin_amdgcn_raw_buffer_load_b128(r, at(bytes, ok), 0, 0);
    }
    __device__ inline f32x4 loadf(uint32_t bytes, bool ok) const
    {
        const u32x4 v = load16(bytes, ok);
        f32x4 f;
        __builtin_memcpy(&f, &v, 16);
        return f;
    }
    __device__ inline float load1(uint32_t bytes, bool ok) const
    {
        return __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(r, at(bytes, ok), 0, 0));
    }
    // four elements of E
    template <typename E> __device__ inline void store(f32x4 v, uint32_t bytes, bool ok) const
    {
        if constexpr (sizeof(E) == 4) {
            u32x4 u;
            __builtin_memcpy(&u, &v, 16);
            __builtin_amdgcn_raw_buffer_store_b128(u, r, at(bytes, ok), 0, 0);
        } else {
            E e[4] = {to_elem<E>(v[0]), to_elem<E>(v[1]), to_elem<E>(v[2]), to_elem<E>(v[3])};
            u32x2 u;
            __builtin_memcpy(&u, e, 8);
            __builtin_amdgcn_raw_buffer_store_b64(u, r, at(bytes, ok), 0, 0);
        }
    }
};

// A [NR][D] tile split into 16-byte chunks over NTH threads (chunk idx =
// tid + h * NTH is row idx / CPR), fetched from global memory into registers
// and later staged into a row-major LDS tile.  Rows r >= `valid` are zero.
template <typename T, int NR, int D, int NTH> struct TileChunks {
    static constexpr int V = 16 / (int)sizeof(T), CPR = D / V, CH = NR * CPR / NTH;
    static_assert(NR * CPR % NTH == 0, "whole chunks per thread");
    u32x4 c[CH];

    // (columns >= dcols, a multiple of V, are zero as well)
    template <typename RowPtr> __device__ inline void fetch(RowPtr rowptr, int valid, int tid, int dcols = D)
    {
#pragma unroll
        for (int h = 0; h < CH; ++h) {
            const int idx = tid + h * NTH, r = idx / CPR, col = (idx % CPR) * V;
            c[h] = u32x4{0u, 0u, 0u, 0u};
            if (r < valid && col < dcols) c[h] = *reinterpret_cast<const u32x4 *>(rowptr(r) + col);
        }
    }

    template <int LDR> __device__ inline void stage(T *sRow, int tid) const
    {
#pragma unroll
        for (int h = 0; h < CH; ++h) {
            const int idx = tid + h * NTH, r = idx / CPR, col = (idx % CPR) * V;
            *reinterpret_cast<u32x4 *>(sRow + r * LDR + col) = c[h];
        }
    }

    // stage(), with rows >= valid written as zero whatever was fetched
    template <int LDR> __device__ inline void stage(T *sRow, int tid, int valid) const
    {
#pragma unroll
        for (int h = 0; h < CH; ++h) {
            const int idx = tid + h * NTH, r = idx / CPR, col = (idx % CPR) * V;
            *reinterpret_cast<u32x4 *>(sRow + r * LDR + col) = r < valid ? c[h] : u32x4{0u, 0u, 0u, 0u};
        }
    }
};

// Lane 16g + c receives X[x0 + 4g + q][c0 + c], q = 0..3, from the row-major
// LDS matrix X (row stride ld elements): the MFMA operand of a product that
// contracts over the rows of X, in the score tiles' slot order.
template <typename T>
__device__ inline typename Mma<T>::frag4 rows4(const T *X, int ld, int x0, int c0, int lane)
{
    const int g = lane >> 4, p = lane & 15;
    const T *src = X + (x0 + 4 * g + (p >> 2)) * ld + c0 + 4 * (p & 3);
    const s16x4 raw = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4 *)(src));
    typename Mma<T>::frag4 out;
    __builtin_memcpy(&out, &raw, 8);
    return out;
}

// B-operand fragments of one 16-row block of a row-major [*, D] matrix:
// lane 16g + c holds row c's elements [KC*cc + KPL*g, +KPL) for every chunk cc.
template <typename T, int D> struct RowFrags {
    using M = Mma<T>;
    typename M::frag f[D / M::KC];
    // from global memory (row == nullptr: a zero row)
    // (columns >= dcols: zero; dcols is a multiple of KPL)
    __device__ inline void load(const T *row, int g, int dcols = D)
    {
#pragma unroll
        for (int c = 0; c < D / M::KC; ++c) {
            if (row && c * M::KC + g * M::KPL < dcols) {
                f[c] = *reinterpret_cast<const typename M::frag *>(row + c * M::KC + g * M::KPL);
            } else {
                f[c] = typename M::frag{};
            }
        }
    }

    // Zero the row when `drop` (a register select: no wait on anything else).
    __device__ inline void clear_if(bool drop)
    {
#pragma unroll
        for (int c = 0; c < D / M::KC; ++c) f[c] = drop ? typename M::frag{} : f[c];
    }
};

// acc = A[r0 + 0..15][0..D) * B-fragments^T : one 16x16 tile of a score product.
// sA_row points to row (r0 + lane%16) of the row-major LDS copy of A.
template <typename T, int D>
__device__ inline f32x4 gemm_scores(const T *sA_row, const RowFrags<T, D> &bf, int g)
{
    using M = Mma<T>;
    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int c = 0; c < D / M::KC; ++c) {
        const typename M::frag a = *reinterpret_cast<const typename M::frag *>(sA_row + c * M::KC + g * M::KPL);
        acc = M::mma(a, bf.f[c], acc);
    }
    return acc;
}

// Operand fragments covering NT 16-wide tiles of a contraction index, in the
// tile-pair slot order: chunk c holds tiles 2c (slots 0..3) and 2c+1 (slots
// 4..7); an odd last tile is a 4-slot fragment.  fp32 keeps one value per
// (tile, slot) for the 16x16x4 instruction.
template <typename T, int NT, bool IS_F32 = std::is_same<T, float>::value> struct ProbFrags;

template <typename T, int NT> struct ProbFrags<T, NT, false> {
    using M = Mma<T>;
    static constexpr int NC = NT / 2;
    typename M::frag f[NC > 0 ? NC : 1];
    typename M::frag4 f4;
    // from score tiles in registers (lane holds 4 rows of each tile)
    __device__ inline void pack(const f32x4 *p)
    {
#pragma unroll
        for (int c = 0; c < NC; ++c) {
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                f[c][q] = to_elem<T>(p[2 * c][q]);
                f[c][4 + q] = to_elem<T>(p[2 * c + 1][q]);
            }
        }
        if constexpr (NT % 2 == 1) {
#pragma unroll
            for (int q = 0; q < 4; ++q) f4[q] = to_elem<T>(p[NT - 1][q]);
        }
    }
    // from a row-major LDS matrix X whose rows are the contraction index
    __device__ inline void gather(const T *X, int ld, int c0, int lane)
    {
#pragma unroll
        for (int c = 0; c < NC; ++c) {
            const typename M::frag4 lo = rows4<T>(X, ld, 32 * c, c0, lane);
            const typename M::frag4 hi = rows4<T>(X, ld, 32 * c + 16, c0, lane);
            f[c] = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
        }
        if constexpr (NT % 2 == 1) f4 = rows4<T>(X, ld, 16 * (NT - 1), c0, lane);
    }
};

template <typename T, int NT> struct ProbFrags<T, NT, true> {
    f32x4 p[NT];
    __device__ inline void pack(const f32x4 *src)
    {
#pragma unroll
        for (int t = 0; t < NT; ++t) p[t] = src[t];
    }
};

// acc[r][col] = sum_x X[x][c0 + r] * B[x][col] over NT 16-wide tiles of x, for
// r = 0..15: one 16x16 tile of an aggregation product.  X is a row-major LDS
// matrix whose rows are the contraction index; B is given as fragments.
template <typename T, int NT>
__device__ inline f32x4 gemm_aggregate(const T *X, int ld, int c0, const ProbFrags<T, NT> &pf, int lane)
{
    using M = Mma<T>;
    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
    if constexpr (std::is_same<T, float>::value) {
        const int g = lane >> 4, c = lane & 15;
#pragma unroll
        for (int t = 0; t < NT; ++t) {
#pragma unroll
            for (int q = 0; q < 4; ++q) acc = M::mma(X[(16 * t + 4 * g + q) * ld + c0 + c], pf.p[t][q], acc);
        }
    } else {
#pragma unroll
        for (int c = 0; c < NT / 2; ++c) {
            const typename M::frag4 lo = rows4<T>(X, ld, 32 * c, c0, lane);
            const typename M::frag4 hi = rows4<T>(X, ld, 32 * c + 16, c0, lane);
            acc = M::mma(__builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7), pf.f[c], acc);
        }
        if constexpr (NT % 2 == 1) acc = M::mma4(rows4<T>(X, ld, 16 * (NT - 1), c0, lane), pf.f4, acc);
    }
    return acc;
}

// acc[r][col] = sum_x B[x][col] for every r: the column sums of the operand
// given as fragments (an all-ones A operand).
template <typename T, int NT>
__device__ inline f32x4 gemm_colsum(const ProbFrags<T, NT> &pf)
{
    using M = Mma<T>;
    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
    typename M::frag ones;
    typename M::frag4 ones4;
#pragma unroll
    for (int q = 0; q < 8; ++q) ones[q] = to_elem<T>(1.0f);
#pragma unroll
    for (int q = 0; q < 4; ++q) ones4[q] = to_elem<T>(1.0f);
#pragma unroll
    for (int c = 0; c < NT / 2; ++c) acc = M::mma(ones, pf.f[c], acc);
    if constexpr (NT % 2 == 1) acc = M::mma4(ones4, pf.f4, acc);
    return acc;
}

// Row tiles per wave and waves per workgroup of a 16-bit unit of NT 16-row
// tiles: one tile a wave.  MA_ROW_TILES = 2 gives a wave two from 4 tiles up, so
// that every operand fragment read from LDS feeds two MFMAs.
#ifndef MA_ROW_TILES
#define MA_ROW_TILES 1
#endif
template <int NT> struct Split {
    static constexpr int RT = (NT >= 4 && MA_ROW_TILES >= 2) ? 2 : 1;
    static constexpr int W = NT / RT;
};

// acc[r] = A[r0 + 0..15][0..D) * bf[r]^T for RT row blocks sharing the A
// fragments (read once from LDS).  sA_row points to row (r0 + lane%16).
template <typename T, int D, int RT>
__device__ inline void gemm_scores_rt(const T *sA_row, const RowFrags<T, D> *bf, f32x4 *acc, int g)
{
    using M = Mma<T>;
#pragma unroll
    for (int r = 0; r < RT; ++r) acc[r] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int c = 0; c < D / M::KC; ++c) {
        const typename M::frag a = *reinterpret_cast<const typename M::frag *>(sA_row + c * M::KC + g * M::KPL);
#pragma unroll
        for (int r = 0; r < RT; ++r) acc[r] = M::mma(a, bf[r].f[c], acc[r]);
    }
}

// acc[r][row][col] = sum_x X[x][c0 + row] * B_r[x][col] for RT operands B_r
// given as fragments, sharing the A fragments read from LDS.
template <typename T, int NT, int RT>
__device__ inline void gemm_aggregate_rt(const T *X, int ld, int c0, const ProbFrags<T, NT> *pf, f32x4 *acc,
                                         int lane)
{
    using M = Mma<T>;
#pragma unroll
    for (int r = 0; r < RT; ++r) acc[r] = f32x4{0.f, 0.f, 0.f, 0.f};
    if constexpr (std::is_same<T, float>::value) {
        const int g = lane >> 4, c = lane & 15;
#pragma unroll
        for (int t = 0; t < NT; ++t) {
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const float a = X[(16 * t + 4 * g + q) * ld + c0 + c];
#pragma unroll
                for (int r = 0; r < RT; ++r) acc[r] = M::mma(a, pf[r].p[t][q], acc[r]);
            }
        }
    } else {
#pragma unroll
        for (int c = 0; c < NT / 2; ++c) {
            const typename M::frag4 lo = rows4<T>(X, ld, 32 * c, c0, lane);
            const typename M::frag4 hi = rows4<T>(X, ld, 32 * c + 16, c0, lane);
            const typename M::frag a = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
#pragma unroll
            for (int r = 0; r < RT; ++r) acc[r] = M::mma(a, pf[r].f[c], acc[r]);
        }
        if constexpr (NT % 2 == 1) {
            const typename M::frag4 a = rows4<T>(X, ld, 16 * (NT - 1), c0, lane);
#pragma unroll
            for (int r = 0; r < RT; ++r) acc[r] = M::mma4(a, pf[r].f4, acc[r]);
        }
    }
}

// Maximum over the softmax index of transposed score tiles (lane holds index
// 16t + 4g + q of row lane%16): in-lane, then across the four lane groups.
// With RAGGED, entries at index >= n are left out.
template <int NT, bool RAGGED>
__device__ inline float tiles_max(const f32x4 *z, int n, int g)
{
    float mx = kMasked;
#pragma unroll
    for (int t = 0; t < NT; ++t) {
#pragma unroll
        for (int q = 0; q < 4; ++q)
            if (!RAGGED || 16 * t + 4 * g + q < n) mx = max_nan(mx, z[t][q]);
    }
    mx = wave_xor_max<16>(mx);
    return wave_xor_max<32>(mx);
}

// 1 / x with the hardware reciprocal (at most 1 ulp from the rounded quotient).
__device__ inline float fast_rcp(float x) { return __builtin_amdgcn_rcpf(x); }

// Whether a softmax is normalised before it feeds a product (4 NT multiplies
// per lane) rather than after it (D / 16 * 4): whichever is fewer.
template <int NT, int D> struct NormFirst {
    static constexpr bool value = 16 * NT < D;
};

__device__ inline float lanegroup_sum(float x)
{
    x = wave_xor_sum<16>(x);
    return wave_xor_sum<32>(x);
}

// Store the 16 x D output tile held as D/16 transposed MFMA tiles (lane holds
// elements 16vt + 4g + q of row lane%16) to the row `row` (nullptr: skip).
// Lanes 16g and 16(g^1) swap halves so that every lane writes 16-byte
// chunks: each row receives 64 contiguous bytes per store instruction.
// Columns >= dcols (a multiple of 16 bytes' worth of elements) are not written.
template <typename T, int D>
__device__ inline void store_row(T *row, const f32x4 *acc, float scale, int lane, int dcols = D)
{
    const int g = lane >> 4;
    if constexpr (std::is_same<T, float>::value) {
        if (row) {
#pragma unroll
            for (int vt = 0; vt < D / 16; ++vt)
                if (16 * vt + 4 * g < dcols) *reinterpret_cast<f32x4 *>(row + 16 * vt + 4 * g) = acc[vt] * scale;
        }
    } else {
        const bool odd = g & 1;
#pragma unroll
        for (int i = 0; i < D / 32; ++i) {
            u32x2 pk[2];
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                T e[4];
#pragma unroll
                for (int q = 0; q < 4; ++q) e[q] = to_elem<T>(acc[2 * i + h][q] * scale);
                __builtin_memcpy(&pk[h], e, 8);
            }
            const u32x2 give = odd ? pk[0] : pk[1];
            u32x2 got;
            got[0] = xor16_value(give[0], odd);
            got[1] = xor16_value(give[1], odd);
            const u32x4 chunk = odd ? u32x4{got[0], got[1], pk[1][0], pk[1][1]}
                                    : u32x4{pk[0][0], pk[0][1], got[0], got[1]};
            const int col = 16 * (2 * i + (odd ? 1 : 0)) + 8 * (g >> 1);
            if (row && col < dcols) *reinterpret_cast<u32x4 *>(row + col) = chunk;
        }
    }
}

// The same 16 x D tile to a row of an LDS matrix: 8 bytes per lane and MFMA
// tile, no exchange between lanes (LDS has no coalescing to serve).
template <typename T, int D> __device__ inline void store_row_lds(T *row, const f32x4 *acc, int lane)
{
    if (!row) return;
    const int g = lane >> 4;
#pragma unroll
    for (int vt = 0; vt < D / 16; ++vt) store4<T>(row + 16 * vt + 4 * g, acc[vt]);
}

struct HeadDims {
    int m, b;          // blocks and block size
    int n;             // rows of q, k, v, out per head, (m - 1) * b < n <= m * b
    int d;             // head dimension of q, k, v, out and of the state rows (<= the tile width D)
    float s_log2e;     // log2(e) / sqrt(d)
    int64_t units;     // work units of a half-step launch (grid size)
    int t = 0, T = 0;  // step of this L half-step (1..T) and the step count, for the objective
    // Per-sequence lengths (batch padding): head bh has lens[bh / H] real
    // rows (clamped to 0..n), or n when lens is null.
    const int *lens = nullptr;
    int H = 1;
    // fp32 L half-step: store alpha_R and c_R of every (k, j) divided by the
    // largest weight L[j][k][l] over l (see LHalf).  Off in the gradient's
    // recompute, whose reverse sweep takes the unscaled states.
    int colnorm = 0;
    // Pre-padded sequences: the kernels run the post-padded problem of the
    // row-reversed tensors, i.e. their row x is row n - 1 - x in memory (for
    // q, k, v and out alike).  The relabelling x -> m b - 1 - x of the padded
    // positions sends block l to m - 1 - l and row j to b - 1 - j: it keeps
    // L^(0) = I and the R and L softmaxes (a permutation of the keys within a
    // block, and of the blocks), and turns padding at the front into padding
    // at the end (Appendix "Padding and Masking").
    int rev = 0;
};

// Row of q, k, v, out in memory for row x (< n) of the kernels' problem.
__device__ inline int64_t mrow(const HeadDims &hd, int64_t x) { return hd.rev ? (int64_t)hd.n - 1 - x : x; }

// Memory rows of the kernels' rows x0 + i*step (i = 0, 1, ...) are
// mrow_u<RV>(x0) + i * rstep<RV>(step): the reversal folds into the first row
// and the sign of the step, so a row address stays one multiply-add.  The
// half-step kernels compile their unit loop with RV = false for calls without
// pre-padding (no reversal at all) and RV = true for the rest.
template <bool RV> __device__ inline int64_t mrow_u(const HeadDims &hd, int64_t x)
{
    return RV ? mrow(hd, x) : x;
}
template <bool RV> __device__ inline int64_t rstep(const HeadDims &hd, int64_t step)
{
    return RV && hd.rev ? -step : step;
}

// The head dimension as the unit code sees it: the compile-time constant DK
// when DK != 0 (the kernels run their unit loop with DK = D when d == D, the
// usual case), else the run-time d.  The row strides of q, k, v, out and of
// the states, and the column bound of their loads and stores, then fold into
// constants where the tile is full.
template <int DK> __device__ inline auto head_dim(int d)
{
    if constexpr (DK != 0)
        return std::integral_constant<int, DK>{};
    else
        return d;
}

// Real rows of head bh.  The kernels read it in fetch() but use it only from
// stage() on: their tile loads take the static bound n, so that they never
// wait for this load, and the rows beyond it are zeroed on their way to LDS.
__device__ inline int live_rows(const HeadDims &hd, int64_t bh)
{
    if (!hd.lens) return hd.n;
    const int len = hd.lens[(int)bh / hd.H];  // bh < 2^31: the grids are checked on the host
    return len < 0 ? 0 : len > hd.n ? hd.n : len;
}

// Real keys of block k of a head with nl real rows: b, fewer in a partly
// padded block, none (<= 0) in a block of padding only.
__device__ inline int block_keys(int b, int nl, int k) { return min(b, nl - k * b); }

// Key blocks holding at least one real key, ceil(nl / b) (m unless the head
// is batch-padded).
__device__ inline int live_blocks(int m, int b, int nl) { return min(m, (nl + b - 1) / b); }

// Tensors and states of one call.  When n < m * b the sequence is taken as
// post-padded with zero rows to N = m * b (Appendix "Padding and Masking"):
// rows >= n of q, k, v are never read (zero is loaded instead), keys >= n are
// masked out of every R softmax, rows >= n of out are never written, and the
// states cover all N rows.  With per-sequence lengths (HeadDims::lens) the
// real rows nl <= n of each head play the part of n: rows nl..n-1 of q, k, v
// may be loaded but are replaced by zero, whole key blocks can be padding
// (such a block gets R = 0, i.e. zero alpha_L, c_L, Y, and no weight in the
// L softmax, Z_L = -inf), and rows nl..n-1 of out are written as zero.
// Layouts (per head):
//   q, k, v, out [B*H][n][d], d <= D (columns d..D-1 of every tile are zero);
//   alpha_R [m][b][d] (row k*b + j), alpha_L and Y [b][m][d] (row j*m + k),
//   c_L [m][b] (written by the R half-step of block k for all j),
//   c_R [b][m] (written by the L half-step of class j for all k).
template <typename T> struct Bufs {
    const T *q, *k, *v;
    T *out;
    T *aR, *aL, *Y;
    float *cR, *cL;
    // Objective shares [B*H][T][b] (nullptr: not requested): after the L update
    // of step t, the sum over the query rows of class j of the logsumexp of the
    // L-update logits (natural units).  Their sum over j is f(M^(t); Q, K).
    float *obj_part = nullptr;
};

// Sum over the 16 rows of a wave (lanes 16g + c, c = 0..15, the four lane
// groups holding the same values): xor steps 8, 4, 2, 1; every lane ends with
// the sum, always in this order.
__device__ inline float rows16_sum(float x)
{
    x += __shfl_xor(x, 8);
    x += __shfl_xor(x, 4);
    x += __shfl_xor(x, 2);
    return x + __shfl_xor(x, 1);
}

// logsumexp (natural units) of a row held as log2-domain logits with maximum
// mx and sum of exp2(logit - mx) = sum.
__device__ inline float row_lse(float mx, float sum) { return kLn2 * (mx + __builtin_amdgcn_logf(sum)); }

}  // namespace ma
