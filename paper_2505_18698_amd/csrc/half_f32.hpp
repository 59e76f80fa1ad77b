// The half-step units for fp32 elements: the units of ma_kernels.hpp (which
// documents their interface) with every operand as three bf16 planes
// (planes.hpp) instead of the fp32 16x16x4 instruction, whose rate bounded
// them (a 128 x 128 x 48 block's R half-step with Y alone is 10 us of it on one
// compute unit).  The tiles are split once, on their way to LDS; a wave splits
// its own rows and probabilities in registers.  V takes K's place in LDS, which
// the planes' size asks for and costs two barriers.  4 heads of 7600 rows
// (60 x 128 blocks, d = 48), us a launch before and now: R (t = 1) 17.0 and
// 12.3, R (last) 23.6 and 15.2, L 11.5 and 9.3, apply 12.7 and 9.4.  What is
// left is latency: 240 or 512 units, one or two a compute unit.  The error
// against 64 bits is 0.73 of what it was (300 drawn calls): a product takes one
// rounding a 32-deep chunk instead of one every 4.
#pragma once

#include "planes.hpp"

namespace ma {

// Rows of fp32 a lane's way (32c + 8g .. + 7 of its row), as loaded.
template <int D> struct RowRaw {
    u32x4 v[D / 32][2];
    __device__ inline void load(const Span &s, int o, bool ok, int g, int d)
    {
#pragma unroll
        for (int c = 0; c < D / 32; ++c) {
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const int col = 32 * c + 8 * g + 4 * h;
                v[c][h] = s.load16((uint32_t)(o + col) * 4, ok && col < d);
            }
        }
    }
    // the planes of chunk c; `drop`: a zero row
    __device__ inline void planes(int c, bool drop, bf16x8 (&f)[3]) const
    {
        float x[8];
        __builtin_memcpy(x, &v[c][0], 32);
#pragma unroll
        for (int i = 0; i < 8; ++i) x[i] = drop ? 0.f : x[i];
        split<3, 8, Reach::kFinite>(x, f);
    }
};

// Probabilities in score-tile order (lane: 4 values of each 16-wide tile) as
// operands of a product over them.
template <int NT> struct Probs32 {
    static constexpr int KD = NT == 1 ? 16 : 32, NC = NT == 1 ? 1 : NT / 2;
    Frag<KD> f[NC][3];
    __device__ inline void pack(const f32x4 *p)
    {
#pragma unroll
        for (int c = 0; c < NC; ++c) {
            float x[KD / 4];
#pragma unroll
            for (int i = 0; i < KD / 4; ++i) x[i] = p[(KD / 16) * c + i / 4][i % 4];
            split<3, KD / 4, Reach::kUnit>(x, f[c]);
        }
    }
    // out[r][col] = sum_x X[x][c0 + r] p[x][col]: X's planes in LDS, rows the contraction index
    __device__ inline f32x4 aggregate(const __bf16 *X, int plane, int ld, int c0, int lane) const
    {
        f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int c = 0; c < NC; ++c) {
            Frag<KD> a[3];
            read_cols<KD, 3>(X, plane, ld, KD * c, c0, lane, a);
            mma_planes(a, f[c], acc);
        }
        return acc;
    }
};

// Scores of a wave's 16 rows (operand rows `bf`) against the rows of X.
template <int NT, int D>
__device__ inline void scores32(const __bf16 *X, int plane, int ld, const bf16x8 (&bf)[D / 32][3], f32x4 (&sc)[NT], int g,
                                int c16)
{
#pragma unroll
    for (int t = 0; t < NT; ++t) {
        Score<true> acc;
#pragma unroll
        for (int c = 0; c < D / 32; ++c) {
            bf16x8 a[3];
            read_chunk<3>(X + (16 * t + c16) * ld, plane, c, g, a);
            acc.add(a, bf[c]);
        }
        sc[t] = acc.value();
    }
}

template <int NB, int D, bool FIRST, bool FINAL, bool RAGGED, bool LENS = false> struct RHalf32 {
    static_assert(!LENS || RAGGED, "per-sequence lengths need the masked softmax");
    static constexpr int NT = NB / 16, W = NT, NTH = 64 * W, LD = D + 16, PLANE = NB * LD;
    static constexpr int LDS_BYTES = 3 * PLANE * 2;  // Kbar[k], then (FINAL) Vbar[k] in its place
    using Tile = Rows<float, 3, NB, D, LD, NTH>;
    using VTile = Rows<float, 3, NB, D, LD, NTH, Reach::kInf>;

    struct Regs {
        Tile kt;
        VTile vt;
        RowRaw<D> row;  // row j of alpha_R[k] (of Q when FIRST)
        float cr;
        int nl, row0;   // real rows of the head, first key row k*b (LENS)
    };

    template <int DK, bool RV>
    __device__ static void fetch(const Bufs<float> &p, const HeadDims &hd, int64_t bh, int k, int tid, Regs &gr)
    {
        if constexpr (LENS) {
            gr.nl = live_rows(hd, bh);
            gr.row0 = k * hd.b;
        }
        const int m = hd.m, b = hd.b, d = head_dim<DK>(hd.d), kv = block_keys(b, hd.n, k);  // rows in memory
        const int64_t N = (int64_t)m * b, hoff = bh * N * d, toff = bh * (int64_t)hd.n * d;
        const int lane = tid & 63, j = (tid >> 6) * 16 + (lane & 15);
        const int r0 = k * b, first = (int)mrow_u<RV>(hd, r0) * d, step = (int)rstep<RV>(hd, 1) * d;
        if constexpr (FIRST)
            gr.row.load(Span(p.q + toff), first + j * step, j < kv, lane >> 4, d);
        else
            gr.row.load(Span(p.aR + hoff), (r0 + j) * d, j < b, lane >> 4, d);
        gr.cr = 1.0f;
        if constexpr (!FIRST) gr.cr = Span(p.cR + bh * N).load1((uint32_t)(j * m + k) * 4, j < b);
        gr.kt.fetch(p.k + toff, step, kv, d, tid, first);
        if constexpr (FINAL) gr.vt.fetch(p.v + toff, step, kv, d, tid, first);
    }

    template <typename U> __device__ static void clear(U &t, int valid, int tid)
    {
#pragma unroll
        for (int h = 0; h < Tile::CH; ++h)
            if ((tid + h * NTH) / Tile::CPR >= valid) t.c[h] = u32x4{0u, 0u, 0u, 0u};
    }

    __device__ static void stage(const HeadDims &, Regs &gr, char *lds, int tid)
    {
        if constexpr (LENS) clear(gr.kt, gr.nl - gr.row0, tid);  // keys >= nl: zero
        gr.kt.stage(reinterpret_cast<__bf16 *>(lds), tid);
    }

    // After stage() and a barrier.
    template <int DK, bool RV>
    __device__ static void compute(const Bufs<float> &p, const HeadDims &hd, int64_t bh, int k, Regs &gr, char *lds, int tid)
    {
        __bf16 *Ks = reinterpret_cast<__bf16 *>(lds);
        // keys >= kv: padding, masked (omega); kv <= 0: padding only, R = 0
        const int m = hd.m, b = hd.b, d = head_dim<DK>(hd.d), kv = block_keys(b, LENS ? gr.nl : hd.n, k);
        const int64_t N = (int64_t)m * b;
        const int lane = tid & 63, g = lane >> 4, c16 = lane & 15, j = (tid >> 6) * 16 + c16;
        const float rs = (FIRST || j >= b) ? hd.s_log2e : hd.s_log2e * fast_rcp(fmaxf(gr.cr, kTiny));
        bf16x8 bf[D / 32][3];
#pragma unroll
        for (int c = 0; c < D / 32; ++c) gr.row.planes(c, FIRST && LENS && j >= kv, bf[c]);
        f32x4 sc[NT];  // lane holds S'[i = 16t + 4g + qq][j]
        scores32<NT, D>(Ks, PLANE, LD, bf, sc, g, c16);
        const float nb = -tiles_max<NT, RAGGED>(sc, kv, g) * rs;
        float sum = 0.f, t2 = 0.f;
#pragma unroll
        for (int t = 0; t < NT; ++t) {
#pragma unroll
            for (int qq = 0; qq < 4; ++qq) {
                const float u = __builtin_fmaf(sc[t][qq], rs, nb);
                float e = __builtin_amdgcn_exp2f(u);
                if (RAGGED && 16 * t + 4 * g + qq >= kv) e = 0.f;
                const bool first = t == 0 && qq == 0;  // the sums start at their first term
                sum = first ? e : sum + e;
                t2 = first ? e * u : __builtin_fmaf(e, u, t2);
                sc[t][qq] = e;
            }
        }
        sum = lanegroup_sum(sum);
        t2 = lanegroup_sum(t2);
        const bool live = !LENS || kv > 0;
        const float inv = live ? fast_rcp(sum) : 0.f;
        // c_L = sum_i R log R = sum_i R (Z - max) - log(sum)   (natural-log units)
        if (g == 0 && j < b)
            p.cL[bh * N + (int64_t)k * b + j] = live ? kLn2 * (t2 * inv - __builtin_amdgcn_logf(sum)) : 0.f;
        Probs32<NT> pf;
        pf.pack(sc);  // unnormalised exp2 values, the row sum is divided out below
        f32x4 out[D / 16];
#pragma unroll
        for (int v = 0; v < D / 16; ++v) out[v] = pf.aggregate(Ks, PLANE, LD, 16 * v, lane);
        store_row<float, D>(j < b ? p.aL + bh * N * d + ((int64_t)j * m + k) * d : nullptr, out, inv, lane, d);
        if constexpr (FINAL) {
            __syncthreads();
            if constexpr (LENS) clear(gr.vt, gr.nl - gr.row0, tid);
            gr.vt.stage(Ks, tid);
            __syncthreads();
#pragma unroll
            for (int v = 0; v < D / 16; ++v) out[v] = pf.aggregate(Ks, PLANE, LD, 16 * v, lane);
            store_row<float, D>(j < b ? p.Y + bh * N * d + ((int64_t)j * m + k) * d : nullptr, out, inv, lane, d);
        }
    }
};

// What the two L units share: alpha_L[j] in LDS, a wave's 16 query rows.
template <int NM, int D, bool RAGGED, bool LENS> struct LBase32 {
    static constexpr int NT = NM / 16, W = NT, NTH = 64 * W, LD = D + 16, PLANE = NM * LD;
    using Tile = Rows<float, 3, NM, D, LD, NTH>;
    // alpha_L[j], which only the scores read: with one wave straight into its
    // registers.  Through LDS (15.4 KB a workgroup instead of 9.3 and 7.7) ten
    // waves shared a compute unit, fewer than the registers allow: 1865 heads of
    // 2 x 63 rows, d = 16: apply 204 -> 125 us; 232 heads of 2 x 123, d = 64: L
    // 49.2 -> 30.1, apply 51.6 -> 32.7; 1024 heads of 16 x 32: L 90 -> 84, apply
    // 131 -> 119; 64 such heads 8.5 and 10.1 either way.
    static constexpr bool DIRECT = NT == 1;
    using ATile = typename std::conditional<DIRECT, RowRaw<D>, Tile>::type;
    static constexpr int A_BYTES = DIRECT ? 0 : 3 * PLANE * 2;

    __device__ static void fetch_a(const Bufs<float> &p, int64_t hoff, int j, int m, int d, int tid, ATile &at)
    {
        const float *base = p.aL + hoff + (int64_t)j * m * d;
        const int r = tid & 15;
        if constexpr (DIRECT)
            at.load(Span(base), r * d, r < m, tid >> 4, d);
        else
            at.fetch(base, d, m, d, tid);
    }
    using YTile = Rows<float, 3, NM, D, LD, NTH, Reach::kInf>;

    // Z (log2 units) of the wave's rows: lane holds k = 16t + 4g + qq of row l = 16 wave + c16.
    __device__ static void logits(const HeadDims &hd, const ATile &at, const __bf16 *As, const float *cLs,
                                  const bf16x8 (&bf)[D / 32][3], f32x4 (&sc)[NT], int g, int c16)
    {
        if constexpr (DIRECT) {
            Score<true> acc;
#pragma unroll
            for (int c = 0; c < D / 32; ++c) {
                bf16x8 a[3];
                at.planes(c, false, a);
                acc.add(a, bf[c]);
            }
            sc[0] = acc.value();
        } else {
            scores32<NT, D>(As, PLANE, LD, bf, sc, g, c16);
        }
#pragma unroll
        for (int t = 0; t < NT; ++t) {
            const f32x4 bias = *reinterpret_cast<const f32x4 *>(cLs + 16 * t + 4 * g);
#pragma unroll
            for (int qq = 0; qq < 4; ++qq) sc[t][qq] = __builtin_fmaf(sc[t][qq], hd.s_log2e, -bias[qq]);
        }
    }
    // ... to exp2(Z - max); returns the sum
    __device__ static float softmax(f32x4 (&sc)[NT], int mk, int g, float &mx)
    {
        mx = tiles_max<NT, RAGGED>(sc, mk, g);
        float sum = 0.f;
#pragma unroll
        for (int t = 0; t < NT; ++t) {
#pragma unroll
            for (int qq = 0; qq < 4; ++qq) {
                float e = __builtin_amdgcn_exp2f(sc[t][qq] - mx);
                if (RAGGED && 16 * t + 4 * g + qq >= mk) e = 0.f;
                sum = (t == 0 && qq == 0) ? e : sum + e;
                sc[t][qq] = e;
            }
        }
        return lanegroup_sum(sum);
    }
    // The objective share of a class: its rows' logsumexps (a workgroup barrier when p.obj_part).
    __device__ static void objective(const Bufs<float> &p, const HeadDims &hd, int64_t bh, int j, float lse, float *objs, int tid)
    {
        if (!p.obj_part) return;
        const float part = rows16_sum(lse);
        if ((tid & 63) == 0) objs[tid >> 6] = part;
        __syncthreads();
        if (tid == 0) {
            float f = 0.f;
            for (int w = 0; w < W; ++w) f += objs[w];
            p.obj_part[(bh * hd.T + hd.t - 1) * hd.b + j] = f;
        }
    }
};

template <int NM, int D, bool RAGGED, bool LENS = false> struct LHalf32 : LBase32<NM, D, RAGGED, LENS> {
    using B = LBase32<NM, D, RAGGED, LENS>;
    using typename B::Tile;
    static constexpr int NT = B::NT, W = B::W, NTH = B::NTH, LD = B::LD, PLANE = B::PLANE, LDP = NM + 8;
    // Qbar[j]; alpha_L[j], then P in fp32
    static constexpr int Q_BYTES = 3 * PLANE * 2, P_BYTES = NM * LDP * 4, AP_BYTES = B::A_BYTES > P_BYTES ? B::A_BYTES : P_BYTES;
    static constexpr int LDS_BYTES = Q_BYTES + AP_BYTES + NM * 4 + W * 4;

    struct Regs {
        Tile qt;
        typename B::ATile at;
        float cl;
        int nl, j;
    };

    template <int DK, bool RV>
    __device__ static void fetch(const Bufs<float> &p, const HeadDims &hd, int64_t bh, int j, int tid, Regs &gr)
    {
        const int m = hd.m, b = hd.b, d = head_dim<DK>(hd.d);
        const int64_t N = (int64_t)m * b;
        if constexpr (LENS) {
            gr.nl = live_rows(hd, bh);
            gr.j = j;
        }
        const int ml = (hd.n - j + b - 1) / b;  // rows l of class j in memory: l*b + j < n
        gr.qt.fetch(p.q + bh * (int64_t)hd.n * d, (int)rstep<RV>(hd, b) * d, ml, d, tid, (int)mrow_u<RV>(hd, j) * d);
        B::fetch_a(p, bh * N * d, j, m, d, tid, gr.at);
        gr.cl = tid < m ? p.cL[bh * N + (int64_t)tid * b + j] : 0.f;
    }

    __device__ static void stage(const HeadDims &hd, Regs &gr, char *lds, int tid)
    {
        if constexpr (LENS) {  // real rows l of class j: l*b + j < nl
            const int ml = (gr.nl - gr.j + hd.b - 1) / hd.b;
#pragma unroll
            for (int h = 0; h < Tile::CH; ++h)
                if ((tid + h * NTH) / Tile::CPR >= ml) gr.qt.c[h] = u32x4{0u, 0u, 0u, 0u};
        }
        gr.qt.stage(reinterpret_cast<__bf16 *>(lds), tid);
        if constexpr (!B::DIRECT) gr.at.stage(reinterpret_cast<__bf16 *>(lds + Q_BYTES), tid);
        if (tid < NM) reinterpret_cast<float *>(lds + Q_BYTES + AP_BYTES)[tid] = gr.cl * kLog2e;
    }

    // After stage() and a barrier.
    template <int DK, bool RV>
    __device__ static void compute(const Bufs<float> &p, const HeadDims &hd, int64_t bh, int j, Regs &gr, char *lds, int tid)
    {
        const __bf16 *Qs = reinterpret_cast<const __bf16 *>(lds), *As = reinterpret_cast<const __bf16 *>(lds + Q_BYTES);
        float *Ps = reinterpret_cast<float *>(lds + Q_BYTES);
        float *cLs = reinterpret_cast<float *>(lds + Q_BYTES + AP_BYTES);
        const int m = hd.m, b = hd.b, d = head_dim<DK>(hd.d);
        const int64_t N = (int64_t)m * b;
        const int lane = tid & 63, g = lane >> 4, c16 = lane & 15, wave = tid >> 6, l = wave * 16 + c16;
        const int mk = LENS ? live_blocks(m, b, gr.nl) : m;  // blocks k >= mk: no real key
        f32x4 sc[NT];
        {
            bf16x8 bf[D / 32][3];
#pragma unroll
            for (int c = 0; c < D / 32; ++c) read_chunk<3>(Qs + l * LD, PLANE, c, g, bf[c]);
            B::logits(hd, gr.at, As, cLs, bf, sc, g, c16);
        }
        const bool logp = hd.colnorm;  // P holds log2 L (below)
        f32x4 zk[NT];
#pragma unroll
        for (int t = 0; t < NT; ++t) zk[t] = sc[t];
        float mx;
        const float sum = B::softmax(sc, mk, g, mx);
        // tile rows l >= m carry no weight, nor does a head without a real key
        const bool live = l < m && (!LENS || mk > 0);
        const float inv = live ? fast_rcp(sum) : 0.f;
        const float lz = live ? mx + __builtin_amdgcn_logf(sum) : 0.f;  // log2 of the row normaliser
        B::objective(p, hd, bh, j, live ? row_lse(mx, sum) : 0.f, cLs + NM, tid);
        __syncthreads();  // every wave is done reading alpha_L
        // P[l][k] into the alpha_L space: L[j][k][l], or with logp its log2 (kMasked where L is zero)
#pragma unroll
        for (int t = 0; t < NT; ++t) {
            f32x4 y;
#pragma unroll
            for (int qq = 0; qq < 4; ++qq) {
                const bool on = inv != 0.f && (!RAGGED || 16 * t + 4 * g + qq < mk);
                y[qq] = !logp ? sc[t][qq] * inv : on ? zk[t][qq] - lz : kMasked;
            }
            *reinterpret_cast<f32x4 *>(Ps + l * LDP + 16 * t + 4 * g) = y;
        }
        __syncthreads();
        // key-block columns k = 16 wave + c16
        const int k = l;
        f32x4 w[NT];
#pragma unroll
        for (int t = 0; t < NT; ++t) {
#pragma unroll
            for (int qq = 0; qq < 4; ++qq) w[t][qq] = Ps[(16 * t + 4 * g + qq) * LDP + k];
        }
        // Column k of L divided by its largest entry: w[l] = 2^(log2 L[j][k][l] - max_l log2 L),
        // so c_R and alpha_R are the eq. beta_r sums times one positive factor per (k, j),
        // which eq. R_update (beta_R / c_R) does not see.  The largest weight is 1, so a
        // column whose weights all lie far below 1 keeps them instead of underflowing.
        if (logp) {
            float mxc = kMasked;
#pragma unroll
            for (int t = 0; t < NT; ++t) {
#pragma unroll
                for (int qq = 0; qq < 4; ++qq) mxc = max_nan(mxc, w[t][qq]);
            }
            mxc = wave_xor_max<32>(wave_xor_max<16>(mxc));
            const bool any = mxc > 0.5f * kMasked;
#pragma unroll
            for (int t = 0; t < NT; ++t) {
#pragma unroll
                for (int qq = 0; qq < 4; ++qq) w[t][qq] = any ? __builtin_amdgcn_exp2f(w[t][qq] - mxc) : 0.f;
            }
        }
        float cs = 0.f;  // c_R[k][j] = sum_l L[j][k][l] (times the factor)
#pragma unroll
        for (int t = 0; t < NT; ++t) cs += (w[t][0] + w[t][1]) + (w[t][2] + w[t][3]);
        cs = lanegroup_sum(cs);
        if (g == 0 && k < m) p.cR[bh * N + (int64_t)j * m + k] = cs;
        Probs32<NT> pf;
        pf.pack(w);
        f32x4 out[D / 16];
#pragma unroll
        for (int v = 0; v < D / 16; ++v) out[v] = pf.aggregate(Qs, PLANE, LD, 16 * v, lane);
        store_row<float, D>(k < m ? p.aR + bh * N * d + ((int64_t)k * b + j) * d : nullptr, out, 1.0f, lane, d);
    }
};

template <int NM, int D, bool RAGGED, bool LENS = false> struct Apply32 : LBase32<NM, D, RAGGED, LENS> {
    using B = LBase32<NM, D, RAGGED, LENS>;
    using typename B::Tile;
    static constexpr int NT = B::NT, W = B::W, NTH = B::NTH, LD = B::LD, PLANE = B::PLANE;
    static constexpr int Y_BYTES = 3 * PLANE * 2, LDS_BYTES = B::A_BYTES + Y_BYTES + NM * 4 + W * 4;  // alpha_L[j], Y[j]

    struct Regs {
        typename B::ATile at;
        typename B::YTile yt;
        float cl;
        RowRaw<D> row;  // row l of Qbar[j]
        int nl;
    };

    template <int DK, bool RV>
    __device__ static void fetch(const Bufs<float> &p, const HeadDims &hd, int64_t bh, int j, int tid, Regs &gr)
    {
        const int m = hd.m, b = hd.b, d = head_dim<DK>(hd.d);
        const int64_t N = (int64_t)m * b, hoff = bh * N * d;
        B::fetch_a(p, hoff, j, m, d, tid, gr.at);
        gr.yt.fetch(p.Y + hoff + (int64_t)j * m * d, d, m, d, tid);
        const int l = (tid >> 6) * 16 + (tid & 15);
        gr.row.load(Span(p.q + bh * (int64_t)hd.n * d), ((int)mrow_u<RV>(hd, j) + l * (int)rstep<RV>(hd, b)) * d, l * b + j < hd.n,
                    (tid & 63) >> 4, d);  // Qbar[j][l]; zero if padded
        gr.cl = tid < m ? p.cL[bh * N + (int64_t)tid * b + j] : 0.f;
        if constexpr (LENS) gr.nl = live_rows(hd, bh);
    }

    __device__ static void stage(const HeadDims &, Regs &gr, char *lds, int tid)
    {
        if constexpr (!B::DIRECT) gr.at.stage(reinterpret_cast<__bf16 *>(lds), tid);
        gr.yt.stage(reinterpret_cast<__bf16 *>(lds + B::A_BYTES), tid);
        if (tid < NM) reinterpret_cast<float *>(lds + B::A_BYTES + Y_BYTES)[tid] = gr.cl * kLog2e;
    }

    // After stage() and a barrier.
    template <int DK, bool RV>
    __device__ static void compute(const Bufs<float> &p, const HeadDims &hd, int64_t bh, int j, Regs &gr, char *lds, int tid)
    {
        const __bf16 *As = reinterpret_cast<const __bf16 *>(lds), *Ys = reinterpret_cast<const __bf16 *>(lds + B::A_BYTES);
        float *cLs = reinterpret_cast<float *>(lds + B::A_BYTES + Y_BYTES);
        const int m = hd.m, b = hd.b, d = head_dim<DK>(hd.d), nl = LENS ? gr.nl : hd.n;
        const int lane = tid & 63, g = lane >> 4, c16 = lane & 15, l = (tid >> 6) * 16 + c16;
        const int mk = LENS ? live_blocks(m, b, nl) : m;  // blocks k >= mk: no real key
        const int row = l * b + j;
        bf16x8 bf[D / 32][3];
#pragma unroll
        for (int c = 0; c < D / 32; ++c) gr.row.planes(c, LENS && row >= nl, bf[c]);
        f32x4 sc[NT];
        B::logits(hd, gr.at, As, cLs, bf, sc, g, c16);
        float mx;
        const float sum = B::softmax(sc, mk, g, mx);
        const bool any = !LENS || mk > 0;  // a head without a real key has L = 0
        const float inv = any ? fast_rcp(sum) : 0.f;
        B::objective(p, hd, bh, j, (l < m && any) ? row_lse(mx, sum) : 0.f, cLs + NM, tid);
        Probs32<NT> pf;
        pf.pack(sc);  // unnormalised, the row sum is divided out of O below
        f32x4 o[D / 16];
#pragma unroll
        for (int v = 0; v < D / 16; ++v) o[v] = pf.aggregate(Ys, PLANE, LD, 16 * v, lane);
        float *ob = p.out + bh * (int64_t)hd.n * d + mrow_u<RV>(hd, j) * d;  // O[j], row 0 of class j
        const int64_t so = rstep<RV>(hd, b) * d;
        // rows nl..n-1 (batch padding) are written as zero
        store_row<float, D>(row < hd.n ? ob + l * so : nullptr, o, (!LENS || row < nl) ? inv : 0.f, lane, d);
    }
};

}  // namespace ma
