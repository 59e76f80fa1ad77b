// Small heads (m, b <= 16, 16-bit elements): the whole forward pass of one
// head in one workgroup (the fully fused one-head-per-block kernel for short
// sequences of Sec. 4, "Benchmarking"); only Q, K, V and O cross global
// memory.
//
// Block k and class j are units of one 16-row tile, and a wave owns the block
// and the class of its number for the whole head.  Only that wave reads
// Qbar[j] and Vbar[k], so they live in its registers (Qbar[j] as rows for the
// scores and transposed for alpha_R, Vbar[k] transposed for Y).  LDS holds
//   A(j, k)  16 x 16 slots of one row: alpha_R[k][j] before an R half-step (at
//            t = 1 the rows of Q), alpha_L[j][k] after it.  The R half-step of
//            block k reads and writes the slots (*, k), the L half-step of
//            class j the slots (j, *), so both work in place (the L half-step
//            passes its probabilities P[l][k] through there);
//   K[k][i]  Kbar[k]; the last R half-step of block k overwrites its own block
//            with Y[k][j]
// and c_R[k][j], c_L[j][k] in fp32.  Half-steps are separated by workgroup
// barriers.  A wave's LDS accesses take effect in program order, so a unit may
// overwrite what it has read.  The arithmetic of a unit is that of RHalf /
// LHalf / Apply at 16 rows, and so are the bits.
//
// What bounds it: the latency of a head's chain (loads, 2 T dependent phases,
// store), not bytes or instructions, so heads should share a compute unit.
// With Q, K and two state regions all in LDS (148 KB at D = 64) one head
// filled it; two regions (76 KB) and 64 VGPRs a wave let two run side by side:
// 384 heads of 15 x 14 rows (197 real), T = 2: 15.2 -> 13.7 us a call; 16 heads of
// 16 x 16 (one a compute unit either way): 7.9 -> 7.1 us.  Two blocks a wave (8 waves,
// 128 VGPRs) took 15.5 us on the first: a wave's phases double in length.
// Wider tiles (109 and 142 KB) keep one head a compute unit; 512 heads of
// 16 x 16 at d = 72, T = 3, take 27 us against 100 us on the half-steps, which
// pass every state through memory in six launches.
#pragma once

#include "ma_kernels.hpp"

namespace ma {

// Where the gradient's recompute keeps the states (FusedHead's KEEP): those of
// step t `st` elements resp. `cst` floats after those of step t - 1, in the
// layouts of Bufs (alpha_R and c_R from step 2 on).
template <typename T> struct KeptStates {
    T *aR, *aL, *Y;
    float *cR, *cL;
    int64_t st, cst;
};

// KEEP: the states go to memory as well, and O is not formed.
template <typename T, int D, bool RGB, bool RGM, bool LENS = false, bool KEEP = false> struct FusedHead {
    static_assert(!LENS || (RGB && RGM), "per-sequence lengths need the masked softmaxes");
    static_assert(sizeof(T) == 2, "16-bit elements only");
    using M = Mma<T>;
    // Where LDS holds two heads a compute unit (D = 64), a workgroup takes one
    // head: without the loop's values a wave needs 60 VGPRs, and two heads fit the
    // registers without spills (2048 heads of 16 x 16 rows, one step: 53 -> 47 us
    // with lengths; of 15 x 14, 40 -> 37).  Wider tiles hold one head, and a
    // workgroup that loops starts the next sooner than a new one does (2048 heads
    // of 15 x 14 rows, d = 72, T = 1: 52 us against 60).
    static constexpr bool LOOP = D > 64;
    // One head a workgroup: ROW workgroups a row of the grid, as a grid dimension
    // of 1024-thread workgroups ends below 2^22 of them.
    static constexpr int LOG_ROW = 21, ROW = 1 << LOG_ROW;
    static constexpr int NTH = 1024, LD = D + 8, NC = D / M::KC, NV = D / 16;
    // Blocks of 16 slots are BS elements apart: 16 rows plus 16 bytes, so that
    // the 16 lanes reading row r of 16 different blocks hit different LDS banks.
    static constexpr int BS = 16 * LD + 8, REGION = 16 * BS;
    static constexpr int CS = 17;  // row stride (floats) of c_R and c_L: writes along a column avoid bank conflicts
    static constexpr int LDS_BYTES = 2 * REGION * (int)sizeof(T) + 2 * 16 * CS * 4;

    // One unit's share of a head: block k = u and class j = u.
    struct Unit {
        RowFrags<T, D> q;              // rows of Qbar[j]
        typename M::frag4 qt[NV], vt[NV];  // Qbar[j] and Vbar[k] transposed
    };

    struct Ctx {
        T *A, *K;
        float *cRs, *cLs;  // c_R[k][j] at k*CS + j, c_L[j][k] at j*CS + k
        int m, b, n, d, lane, g, c16;  // n: rows of a head in q, k, v, out; d <= D
        int rev;                       // pre-padded: row x in memory at n - 1 - x (HeadDims::rev)
        int nl, mk;        // with per-sequence lengths: real rows of the head being computed, live key blocks
        float s_log2e;
        int64_t bh;        // the head being computed
        int steps;         // T, the step count
        float *obj_part;   // objective shares [B*H][T][b], or nullptr
        KeptStates<T> keep;  // of this head and step (KEEP)
    };

    // The 16 rows of block k of q, k or v in registers, 16-byte chunks in row
    // order over the lanes (whole cache lines an instruction); zero past the
    // block's rows, the head's and the d columns.
    static constexpr int CPR = D / 8, CH = 16 * CPR / 64;
    struct Block {
        u32x4 c[CH];
    };
    __device__ static void load_block(const Ctx &c, const Span &s, int k, Block &f)
    {
#pragma unroll
        for (int h = 0; h < CH; ++h) {
            const int idx = c.lane + 64 * h, r = idx / CPR, col = (idx % CPR) * 8, x = k * c.b + r;
            const int row = c.rev ? c.n - 1 - x : x;
            f.c[h] = s.load16((uint32_t)(row * c.d + col) * 2, k < c.m && r < c.b && x < c.n && col < c.d);
        }
    }
    // ... with rows >= nl cleared, to LDS rows `step` elements apart
    __device__ static void store_block(const Ctx &c, const Block &f, int k, T *X, int step)
    {
#pragma unroll
        for (int h = 0; h < CH; ++h) {
            const int idx = c.lane + 64 * h, r = idx / CPR, col = (idx % CPR) * 8;
            *reinterpret_cast<u32x4 *>(X + r * step + col) =
                (!LENS || k * c.b + r < c.nl) ? f.c[h] : u32x4{0u, 0u, 0u, 0u};
        }
    }

    // The rows of an LDS block, transposed.
    __device__ static void read_cols(const Ctx &c, const T *X, typename M::frag4 (&t)[NV])
    {
#pragma unroll
        for (int v = 0; v < NV; ++v) t[v] = rows4<T>(X, LD, 0, 16 * v, c.lane);
    }

    // R half-step of block k (first: t = 1, c_R = 1; last: also Y).
    __device__ static void r_unit(const Ctx &c, int k, const Unit &un, bool first, bool last)
    {
        const int j = c.c16;
        const bool jv = j < c.b;
        T *row = c.A + j * BS;
        RowFrags<T, D> bf, kf;  // row j of alpha_R[k], row i of Kbar[k]
        bf.load(row + k * LD, c.g);
        kf.load(c.K + k * BS + j * LD, c.g);
        float rs = c.s_log2e;
        if (!first && jv) rs = c.s_log2e * fast_rcp(fmaxf(c.cRs[k * CS + j], kTiny));
        f32x4 sc = {0.f, 0.f, 0.f, 0.f};  // lane holds S'[i = 4g + qq][j]
#pragma unroll
        for (int i = 0; i < NC; ++i) sc = M::mma(kf.f[i], bf.f[i], sc);
        const int kv = block_keys(c.b, LENS ? c.nl : c.n, k);  // keys >= kv: padding, masked (omega); none: R = 0
        const float nb = -tiles_max<1, RGB>(&sc, kv, c.g) * rs;
        float sum = 0.f, t2 = 0.f;
#pragma unroll
        for (int qq = 0; qq < 4; ++qq) {
            const float u = __builtin_fmaf(sc[qq], rs, nb);
            float e = __builtin_amdgcn_exp2f(u);
            if (RGB && 4 * c.g + qq >= kv) e = 0.f;
            sum = qq == 0 ? e : sum + e;
            t2 = qq == 0 ? e * u : __builtin_fmaf(e, u, t2);
            sc[qq] = e;
        }
        sum = lanegroup_sum(sum);
        t2 = lanegroup_sum(t2);
        const bool live = !LENS || kv > 0;
        const float inv = live ? fast_rcp(sum) : 0.f;
        if (c.g == 0 && jv) {
            const float cl = live ? kLn2 * (t2 * inv - __builtin_amdgcn_logf(sum)) : 0.f;
            c.cLs[j * CS + k] = cl;
            if constexpr (KEEP) c.keep.cL[k * c.b + j] = cl;
        }
        static_assert(NormFirst<1, D>::value, "probabilities normalised before the products, as in RHalf");
        sc *= inv;
        ProbFrags<T, 1> pf;
        pf.pack(&sc);
        const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
        const bool on = jv;
        T *Kk = c.K + k * BS;
        f32x4 o[NV];
#pragma unroll
        for (int v = 0; v < NV; ++v) {
            o[v] = M::mma4(rows4<T>(Kk, LD, 0, 16 * v, c.lane), pf.f4, zero);
            if (on && !(KEEP && last)) store4<T>(row + k * LD + 16 * v + 4 * c.g, o[v]);  // alpha_L[j][k]
        }
        if constexpr (KEEP) store_row<T, D>(on ? c.keep.aL + (j * c.m + k) * c.d : nullptr, o, 1.0f, c.lane, c.d);
        if (last) {  // Y[k][j] over Kbar[k] (blocks k >= m stay zero: they meet zero probabilities in the apply)
#pragma unroll
            for (int v = 0; v < NV; ++v) {
                o[v] = M::mma4(un.vt[v], pf.f4, zero);
                if (on && !KEEP) store4<T>(Kk + j * LD + 16 * v + 4 * c.g, o[v]);
            }
            if constexpr (KEEP) store_row<T, D>(on ? c.keep.Y + (j * c.m + k) * c.d : nullptr, o, 1.0f, c.lane, c.d);
        }
    }

    // Scores and softmax over k of class j, query row l = lane % 16
    // (lane holds k = 4g + qq); returns exp2 values and sets inv = 1 / row sum
    // and lse = the row's logsumexp (natural units; 0 for tile rows l >= m).
    __device__ static void l_softmax(const Ctx &c, int j, const Unit &un, f32x4 &sc, float &inv, float &lse)
    {
        f32x4 acc;
        gemm_scores_rt<T, D, 1>(c.A + j * BS + c.c16 * LD, &un.q, &acc, c.g);
#pragma unroll
        for (int qq = 0; qq < 4; ++qq) {
            // entries k >= m hold no c_L (their LDS words are never written);
            // the selects below leave them out of the maximum and the sum
            const float bias = c.cLs[j * CS + 4 * c.g + qq] * kLog2e;
            sc[qq] = __builtin_fmaf(acc[qq], c.s_log2e, -bias);
        }
        const int mk = LENS ? c.mk : c.m;  // blocks k >= mk: no real key
        const float mx = tiles_max<1, RGM>(&sc, mk, c.g);
        float sum = 0.f;
#pragma unroll
        for (int qq = 0; qq < 4; ++qq) {
            float e = __builtin_amdgcn_exp2f(sc[qq] - mx);
            if (RGM && 4 * c.g + qq >= mk) e = 0.f;
            sum = qq == 0 ? e : sum + e;
            sc[qq] = e;
        }
        sum = lanegroup_sum(sum);
        const bool any = !LENS || mk > 0;  // a head without a real key has L = 0
        inv = any ? fast_rcp(sum) : 0.f;
        lse = (c.c16 < c.m && any) ? row_lse(mx, sum) : 0.f;
    }

    // Objective share of class j after the L update of step t (as LHalf / Apply).
    __device__ static void objective_share(const Ctx &c, int j, int t, float lse)
    {
        if (!c.obj_part) return;
        const float part = rows16_sum(lse);
        if (c.lane == 0) c.obj_part[(c.bh * c.steps + t - 1) * c.b + j] = part;
    }

    __device__ static void l_unit(const Ctx &c, int j, int t, const Unit &un)
    {
        const int l = c.c16, k = c.c16;
        float inv, lse;
        f32x4 e;
        l_softmax(c, j, un, e, inv, lse);
        objective_share(c, j, t, lse);
        ProbFrags<T, 1> pf;  // B operand: P[l-slots][k = lane % 16]
        // alpha_L[j] has been read: P[l][k] in its place
        const f32x4 pr = l < c.m ? e * inv : f32x4{0.f, 0.f, 0.f, 0.f};  // padded query rows carry no weight
        store4<T>(c.A + j * BS + l * LD + 4 * c.g, pr);
        pf.gather(c.A + j * BS, LD, 0, c.lane);
        const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
        const f32x4 cs = gemm_colsum<T, 1>(pf);  // c_R[k][j] = sum_l L[j][k][l]
        const bool on = k < c.m;
        if (c.g == 0 && on) {
            c.cRs[k * CS + j] = cs[0];
            if constexpr (KEEP) c.keep.cR[j * c.m + k] = cs[0];
        }
        f32x4 o[NV];
#pragma unroll
        for (int v = 0; v < NV; ++v) {
            o[v] = M::mma4(un.qt[v], pf.f4, zero);
            if (on) store4<T>(c.A + j * BS + k * LD + 16 * v + 4 * c.g, o[v]);  // alpha_R[k][j]
        }
        if constexpr (KEEP) store_row<T, D>(on ? c.keep.aR + (k * c.b + j) * c.d : nullptr, o, 1.0f, c.lane, c.d);
    }

    __device__ static void apply_unit(const Ctx &c, int j, const Unit &un, T *out_h)
    {
        float inv, lse;
        f32x4 e;
        l_softmax(c, j, un, e, inv, lse);
        objective_share(c, j, c.steps, lse);
        const f32x4 pr = e * inv;  // normalised first, as in Apply at 16 rows
        ProbFrags<T, 1> pf;
        pf.pack(&pr);
        f32x4 o[NV];  // O[l*b + j] = sum_k L[j][k][l] Y[k][j]; Y[k][j] is row k of K + j*LD at stride BS
#pragma unroll
        for (int v = 0; v < NV; ++v) o[v] = gemm_aggregate<T, 1>(c.K + j * LD, BS, 16 * v, pf, c.lane);
        const int row = c.c16 * c.b + j;  // rows nl..n-1 (batch padding) are written as zero
        const int64_t mr = c.rev ? (int64_t)c.n - 1 - row : row;
        store_row<T, D>(row < c.n ? out_h + mr * c.d : nullptr, o, (!LENS || row < c.nl) ? 1.0f : 0.f,
                        c.lane, c.d);
    }

    // Head blockIdx.x of row blockIdx.y (LOOP: heads blockIdx.x, blockIdx.x + gridDim.x, ... < BH).
    __device__ static void run(const Bufs<T> &p, const HeadDims &hd, int64_t BH, int T_, const KeptStates<T> &keep,
                               char *lds)
    {
        Ctx c;
        c.A = reinterpret_cast<T *>(lds);
        c.K = c.A + REGION;
        c.cRs = reinterpret_cast<float *>(c.K + REGION);
        c.cLs = c.cRs + 16 * CS;
        c.m = hd.m;
        c.b = hd.b;
        c.n = hd.n;
        c.d = hd.d;
        c.rev = hd.rev;
        c.s_log2e = hd.s_log2e;
        c.steps = T_;
        c.obj_part = p.obj_part;
        const int tid = threadIdx.x, w = __builtin_amdgcn_readfirstlane(tid >> 6);
        c.lane = tid & 63;
        c.g = c.lane >> 4;
        c.c16 = c.lane & 15;

        int64_t bh = blockIdx.x;
        if constexpr (!LOOP) {
            bh += (int64_t)blockIdx.y << LOG_ROW;
            if (bh >= BH) return;
        }
        for (;;) {
            c.bh = bh;
            const int64_t hoff = bh * (int64_t)c.n * c.d;
            const Span qs(p.q + hoff), ks(p.k + hoff), vs(p.v + hoff);
            Unit un;
            {
                Block qb, kb, vb;
                load_block(c, qs, w, qb);
                load_block(c, ks, w, kb);
                load_block(c, vs, w, vb);
                if constexpr (LENS) {
                    // the loads were issued with the static bound n: rows >= nl are zeroed on their way to LDS
                    c.nl = live_rows(hd, bh);
                    c.mk = live_blocks(c.m, c.b, c.nl);
                }
                // Q rows k*b + j into the slots (j, k): alpha_R[k] of t = 1, and the rows l = k of Qbar[j]
                const int k = w;
                T *X = c.K + k * BS;
                store_block(c, qb, k, c.A + k * LD, BS);
                store_block(c, vb, k, X, LD);
                read_cols(c, X, un.vt);
                store_block(c, kb, k, X, LD);
            }
            __syncthreads();
            const T *X = c.A + w * BS;
            un.q.load(X + c.c16 * LD, c.g);
            read_cols(c, X, un.qt);
            __syncthreads();  // the first half-step writes A

            for (int t = 1; t <= T_; ++t) {
                if constexpr (KEEP) {
                    const int64_t rows = bh * c.m * c.b, s0 = (t - 1) * keep.st + rows * c.d, c0 = (t - 1) * keep.cst + rows;
                    c.keep = KeptStates<T>{keep.aR + s0, keep.aL + s0, keep.Y + rows * c.d, keep.cR + c0, keep.cL + c0, 0, 0};
                }
                if (w < c.m) r_unit(c, w, un, t == 1, t == T_);
                if (KEEP && t == T_) break;
                __syncthreads();
                if (t == T_) break;
                if (w < c.b) l_unit(c, w, t, un);
                __syncthreads();
            }
            if (!KEEP && w < c.b) apply_unit(c, w, un, p.out + hoff);
            if constexpr (!LOOP) return;
            bh += gridDim.x;
            if (bh >= BH) return;
            __syncthreads();  // the next head overwrites A and K
        }
    }
};

template <typename T, int D, bool RGB, bool RGM, bool LENS>
__global__ __launch_bounds__(1024, D == 64 ? 8 : 4) void monarch_fused_head(Bufs<T> p, HeadDims hd, int64_t BH, int T_)
{
    using U = FusedHead<T, D, RGB, RGM, LENS>;
    __shared__ __attribute__((aligned(16))) char lds[U::LDS_BYTES];
    U::run(p, hd, BH, T_, KeptStates<T>{}, lds);
}

// The gradient's recompute of small heads: every step's states to memory, as
// whole rows from the registers that hold them.  At D = 64 that takes 66 VGPRs,
// so one head a compute unit; held to 64, with spills, 4 heads of 15 x 14 rows
// take 4% longer a gradient (T = 2) and 2048 heads as long.
template <typename T, int D, bool RGB, bool RGM, bool LENS>
__global__ __launch_bounds__(1024, 4) void monarch_fused_states(Bufs<T> p, HeadDims hd, int64_t BH, int T_, KeptStates<T> keep)
{
    using U = FusedHead<T, D, RGB, RGM, LENS, true>;
    __shared__ __attribute__((aligned(16))) char lds[U::LDS_BYTES];
    U::run(p, hd, BH, T_, keep, lds);
}

}  // namespace ma
