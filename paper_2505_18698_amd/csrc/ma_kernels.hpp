// MonarchAttention forward kernels for CDNA4 (gfx950).
//
// One kernel per half-step of the alternating maximisation (Sec. 3 of the
// paper, eqs. R_update / L_update with beta_r / beta_l), organised as in the
// paper's Implementation paragraph: the factors L and R live only in
// registers and LDS; between launches only the states alpha_R, c_R, alpha_L,
// c_L and Y cross global memory.
//
//   r_half_step<FIRST, FINAL>  one workgroup per (head, key block k):
//        S'[i][j] = Kbar[k][i] . alpha_R[k][j]                (beta_R, MFMA)
//        R[k][j][:] = softmax_i(s * S'[:, j] / c_R[k][j])      (eq. R_update)
//        c_L[j][k] = sum_i R log R,  alpha_L[j][k] = R Kbar[k] (eq. beta_l, MFMA)
//        FINAL: Y[j][k] = R Vbar[k]                            (eq. monarch_multiply)
//   l_half_step                one workgroup per (head, residue class j):
//        S'[k][l] = alpha_L[j][k] . Qbar[j][l]                 (beta_L, MFMA)
//        L[j][:][l] = softmax_k(s * S'[:, l] - c_L[j][:])      (eq. L_update)
//        c_R[k][j] = sum_l L,  alpha_R[k][j] = sum_l L Qbar[j][l]   (eq. beta_r, MFMA)
//   monarch_apply              one workgroup per (head, j): the last L half-step
//        fused with O[l*b + j] = sum_k L[j][k][l] Y[j][k]     (eq. monarch_multiply)
//
// The permutation P is never materialised: Qbar[j][l] is row l*b + j of Q, so
// the L half-step and the apply read (and the apply writes) rows at a stride of
// b rows, each row one contiguous d-element segment.
//
// MFMA use.  Every product is a 16x16 output tile of v_mfma_f32_16x16x{32,16}
// with fp32 accumulation (fp32 elements: as bf16 planes, half_f32.hpp).  Lane l of a wave owns
// output rows 4*(l/16)+q (q = 0..3) of column l%16.  Scores are formed
// transposed (softmax index along the rows of the MFMA tile), so each lane
// holds a whole column slice of one softmax row: the max and sum are an
// in-lane reduction plus two cross-lane steps.  The probabilities left in
// registers feed the second product directly as its B operand: for a chunk of
// 32 contraction indices made of two 16-wide score tiles, lane l's 8 operand
// slots are the 4 rows it holds of each tile.  The A operand of that product
// (a row-major LDS tile whose rows are the contraction index) is read with
// the gfx950 LDS transpose load ds_read_b64_tr_b16, which hands lane 16g + c
// the column c of rows 4g..4g+3 of a 16-row group, i.e. the same slot order.
#pragma once

#include "half_f32.hpp"

namespace ma {

// The work of one unit of each half-step, done by a workgroup of W waves in
// three parts: fetch() issues its global loads into registers, stage() moves
// the tiles into LDS, and compute() (after a barrier) does the rest.  RAGGED:
// the softmax index range (b for R, m for L) is shorter than the padded tile.

// ---------------------------------------------------------------------------------------
// R half-step for (head bh, key block k); each wave owns RT tiles of 16 rows j.
// NB = b rounded up to 16.  FIRST: alpha_R = the rows of Q (L^(0) = I) and
// c_R = 1.  FINAL: also Y.
// ---------------------------------------------------------------------------------------
template <typename T, int NB, int D, bool FIRST, bool FINAL, bool RAGGED, bool LENS = false> struct RHalf {
    static_assert(!LENS || RAGGED, "per-sequence lengths need the masked softmax");
    static constexpr int NT = NB / 16, RT = Split<NT>::RT, W = Split<NT>::W, NTH = 64 * W;
    static constexpr bool NF = NormFirst<NT, D>::value;
    static constexpr int LDK = Ld<T, D>::row;
    static constexpr int LDS_BYTES = (FINAL ? 2 : 1) * NB * LDK * (int)sizeof(T);

    // What a unit reads from global memory, held in registers until staged.
    struct Regs {
        TileChunks<T, NB, D, NTH> kt, vt;  // Kbar[k]; Vbar[k] (FINAL)
        RowFrags<T, D> bf[RT];             // rows j of alpha_R[k] (of Q when FIRST)
        float cr[RT];                      // c_R[k][j] (not FIRST)
        int nl, row0;                      // real rows of the head, first key row k*b (LENS)
    };

    template <int DK, bool RV>
    __device__ static void fetch(const Bufs<T> &p, const HeadDims &hd, int64_t bh, int k, int tid, Regs &gr)
    {
        if constexpr (LENS) {
            gr.nl = live_rows(hd, bh);
            gr.row0 = k * hd.b;
        }
        const int m = hd.m, b = hd.b, kv = block_keys(b, hd.n, k);  // rows in memory
        const auto dd = head_dim<DK>(hd.d);
        const int64_t N = (int64_t)m * b, hoff = bh * N * dd, toff = bh * (int64_t)hd.n * dd;  // states: rows of d
        const int lane = tid & 63, wave = tid >> 6;
        const int64_t r0 = (int64_t)k * b, first = mrow_u<RV>(hd, r0), step = rstep<RV>(hd, 1);
#pragma unroll
        for (int r = 0; r < RT; ++r) {
            const int j = (wave * RT + r) * 16 + (lane & 15);
            const T *row = nullptr;  // alpha_R[k][j]; at t = 1 Q row k*b + j (zero if padding)
            if constexpr (FIRST) {
                if (j < kv) row = p.q + toff + (first + j * step) * dd;
            } else {
                if (j < b) row = p.aR + hoff + (r0 + j) * dd;
            }
            gr.bf[r].load(row, lane >> 4, dd);
            gr.cr[r] = 1.0f;
            if constexpr (!FIRST) {
                if (j < b) gr.cr[r] = p.cR[bh * N + (int64_t)j * m + k];
            }
        }
        // K and V after the alpha_R rows, V last: the scores wait for the rows
        // and K only, and V is staged just before the product that needs it
        const int64_t sd = step * dd;
        const T *kb = p.k + toff + first * dd;
        gr.kt.fetch([=](int r) { return kb + r * sd; }, kv, tid, dd);
        if constexpr (FINAL) {
            const T *vb = p.v + toff + first * dd;
            gr.vt.fetch([=](int r) { return vb + r * sd; }, kv, tid, dd);
        }
    }

    __device__ static void stage(const HeadDims &, const Regs &gr, char *lds, int tid)
    {
        T *Ks = reinterpret_cast<T *>(lds);
        if constexpr (LENS) {  // keys >= nl: zero (they are masked, zero keeps them finite)
            const int kv = gr.nl - gr.row0;
            gr.kt.template stage<LDK>(Ks, tid, kv);
        } else {
            gr.kt.template stage<LDK>(Ks, tid);
        }
    }

    // After stage() and a barrier.
    template <int DK, bool RV>
    __device__ static void compute(const Bufs<T> &p, const HeadDims &hd, int64_t bh, int k, const Regs &gr,
                                   char *lds, int tid)
    {
        T *Ks = reinterpret_cast<T *>(lds);
        T *Vs = Ks + NB * LDK;
        // keys >= kv: padding, masked (omega); kv <= 0: padding only, R = 0
        const int m = hd.m, b = hd.b, kv = block_keys(b, LENS ? gr.nl : hd.n, k);
        const int64_t N = (int64_t)m * b;
        const int lane = tid & 63, wave = tid >> 6;
        const int g = lane >> 4, c16 = lane & 15;
        int jr[RT];
        float rscale[RT];
#pragma unroll
        for (int r = 0; r < RT; ++r) {
            jr[r] = (wave * RT + r) * 16 + c16;
            rscale[r] = (FIRST || jr[r] >= b) ? hd.s_log2e : hd.s_log2e * fast_rcp(fmaxf(gr.cr[r], kTiny));
        }

        RowFrags<T, D> bfq[RT];  // at t = 1 with per-sequence lengths: Q rows beyond the length zeroed
        if constexpr (FIRST && LENS) {
#pragma unroll
            for (int r = 0; r < RT; ++r) {
                bfq[r] = gr.bf[r];
                bfq[r].clear_if(jr[r] >= kv);
            }
        }
        const RowFrags<T, D> *bf = (FIRST && LENS) ? bfq : gr.bf;
        f32x4 sc[RT][NT];  // lane holds S'[i = 16t + 4g + qq][j] of row tile r
#pragma unroll
        for (int t = 0; t < NT; ++t) {
            f32x4 acc[RT];
            gemm_scores_rt<T, D, RT>(Ks + (16 * t + c16) * LDK, bf, acc, g);
#pragma unroll
            for (int r = 0; r < RT; ++r) sc[r][t] = acc[r];
        }
        ProbFrags<T, NT> pf[RT];
        float inv[RT];
#pragma unroll
        for (int r = 0; r < RT; ++r) {
            // Z = s S / c_R in log2 units: u = Z - max Z = S * rs - max S * rs  (rs > 0)
            const float rs = rscale[r];
            const float nb = -tiles_max<NT, RAGGED>(sc[r], kv, g) * rs;
            float sum = 0.f, t2 = 0.f;
#pragma unroll
            for (int t = 0; t < NT; ++t) {
#pragma unroll
                for (int qq = 0; qq < 4; ++qq) {
                    const float u = __builtin_fmaf(sc[r][t][qq], rs, nb);
                    float e = __builtin_amdgcn_exp2f(u);
                    if (RAGGED && 16 * t + 4 * g + qq >= kv) e = 0.f;
                    const bool first = t == 0 && qq == 0;  // the sums start at their first term
                    sum = first ? e : sum + e;
                    t2 = first ? e * u : __builtin_fmaf(e, u, t2);
                    sc[r][t][qq] = e;
                }
            }
            sum = lanegroup_sum(sum);
            t2 = lanegroup_sum(t2);
            const bool live = !LENS || kv > 0;
            inv[r] = live ? fast_rcp(sum) : 0.f;
            // c_L = sum_i R log R = sum_i R (Z - max) - log(sum)   (natural-log units)
            if (g == 0 && jr[r] < b)
                p.cL[bh * N + (int64_t)k * b + jr[r]] =
                    live ? kLn2 * (t2 * inv[r] - __builtin_amdgcn_logf(sum)) : 0.f;
            if constexpr (NF) {
#pragma unroll
                for (int t = 0; t < NT; ++t) sc[r][t] *= inv[r];
                inv[r] = 1.0f;
            }
            pf[r].pack(sc[r]);  // !NF: unnormalised exp2 values, the row sum is divided out below
        }
        f32x4 out[RT][D / 16];
#pragma unroll
        for (int vt = 0; vt < D / 16; ++vt) {
            f32x4 acc[RT];
            gemm_aggregate_rt<T, NT, RT>(Ks, LDK, 16 * vt, pf, acc, lane);
#pragma unroll
            for (int r = 0; r < RT; ++r) out[r][vt] = acc[r];
        }
        const auto dd = head_dim<DK>(hd.d);  // states: rows of d elements
#pragma unroll
        for (int r = 0; r < RT; ++r)  // alpha_L[j][k] (j-major)
            store_row<T, D>(jr[r] < b ? p.aL + bh * N * dd + ((int64_t)jr[r] * m + k) * dd : nullptr, out[r],
                            inv[r], lane, dd);
        if constexpr (FINAL) {
            // Vbar[k], staged here rather than with K: when a workgroup runs a
            // single unit, the scores and softmax overlap V's loads
            if constexpr (LENS)
                gr.vt.template stage<LDK>(Vs, tid, gr.nl - gr.row0);
            else
                gr.vt.template stage<LDK>(Vs, tid);
            __syncthreads();
#pragma unroll
            for (int vt = 0; vt < D / 16; ++vt) {
                f32x4 acc[RT];
                gemm_aggregate_rt<T, NT, RT>(Vs, LDK, 16 * vt, pf, acc, lane);
#pragma unroll
                for (int r = 0; r < RT; ++r) out[r][vt] = acc[r];
            }
#pragma unroll
            for (int r = 0; r < RT; ++r)
                store_row<T, D>(jr[r] < b ? p.Y + bh * N * dd + ((int64_t)jr[r] * m + k) * dd : nullptr, out[r],
                                inv[r], lane, dd);
        }
    }
};

// ---------------------------------------------------------------------------------------
// L half-step (not the last) for (head bh, residue class j).  NM = m rounded
// up to 16.  Wave w first owns RT tiles of 16 query rows l (scores and the
// softmax over k), then, after the probabilities have gone through LDS, RT
// tiles of 16 key-block columns k (c_R and alpha_R).
// ---------------------------------------------------------------------------------------
template <typename T, int NM, int D, bool RAGGED, bool LENS = false> struct LHalf {
    static_assert(!LENS || RAGGED, "per-sequence lengths need the masked softmax");
    static constexpr int NT = NM / 16, RT = Split<NT>::RT, W = Split<NT>::W, NTH = 64 * W;
    // P rows are padded by 8 elements, not the usual 32 bytes: with 16-bit
    // elements, the 16 rows that one P store instruction writes at one
    // column then fall on distinct LDS banks (at 128 rows the L half-step ran
    // 7% faster than with the 32-byte pad; pads of 4 and 24 measured the same).
    static constexpr int LDQ = Ld<T, D>::row, LDP = NM + 8;
    static constexpr int A_ELEMS = NM * LDQ, P_ELEMS = NM * LDP;
    static constexpr int AP_ELEMS = A_ELEMS > P_ELEMS ? A_ELEMS : P_ELEMS;
    static constexpr int LDS_BYTES = (NM * LDQ + AP_ELEMS) * (int)sizeof(T) + NM * 4 + W * 4;

    struct Regs {
        TileChunks<T, NM, D, NTH> qt, at;  // Qbar[j] (rows l), alpha_L[j] (rows k)
        float cl;                          // c_L[k = tid][j]
        int nl, j;                         // real rows of the head, the class (LENS)
    };

    template <int DK, bool RV>
    __device__ static void fetch(const Bufs<T> &p, const HeadDims &hd, int64_t bh, int j, int tid, Regs &gr)
    {
        const int m = hd.m, b = hd.b;
        const int64_t N = (int64_t)m * b;
        if constexpr (LENS) {
            gr.nl = live_rows(hd, bh);
            gr.j = j;
        }
        const int ml = (hd.n - j + b - 1) / b;  // rows l of class j in memory: l*b + j < n
        const auto dd = head_dim<DK>(hd.d);
        const int64_t hoff = bh * N * dd;  // states: rows of d elements
        const T *qb = p.q + bh * (int64_t)hd.n * dd + mrow_u<RV>(hd, j) * dd;  // Qbar[j][0]
        const int64_t sq = rstep<RV>(hd, b) * dd;                           // Qbar[j][l] -> Qbar[j][l + 1]
        const T *al = p.aL + hoff + (int64_t)j * m * dd;
        gr.qt.fetch([=](int l) { return qb + l * sq; }, ml, tid, dd);
        gr.at.fetch([=](int kk) { return al + (int64_t)kk * dd; }, m, tid, dd);
        gr.cl = tid < m ? p.cL[bh * N + (int64_t)tid * b + j] : 0.f;
    }

    __device__ static void stage(const HeadDims &hd, const Regs &gr, char *lds, int tid)
    {
        T *Qs = reinterpret_cast<T *>(lds);
        T *APs = Qs + NM * LDQ;
        if constexpr (LENS)  // real rows l of class j: l*b + j < nl
            gr.qt.template stage<LDQ>(Qs, tid, (gr.nl - gr.j + hd.b - 1) / hd.b);
        else
            gr.qt.template stage<LDQ>(Qs, tid);
        gr.at.template stage<LDQ>(APs, tid);
        if (tid < NM) reinterpret_cast<float *>(APs + AP_ELEMS)[tid] = gr.cl * kLog2e;
    }

    // After stage() and a barrier.
    template <int DK, bool RV>
    __device__ static void compute(const Bufs<T> &p, const HeadDims &hd, int64_t bh, int j, const Regs &gr,
                                   char *lds, int tid)
    {
        T *Qs = reinterpret_cast<T *>(lds);
        T *APs = Qs + NM * LDQ;  // alpha_L, then P
        float *cLs = reinterpret_cast<float *>(APs + AP_ELEMS);
        const int m = hd.m, b = hd.b;
        const int64_t N = (int64_t)m * b;
        const int lane = tid & 63, wave = tid >> 6;
        const int g = lane >> 4, c16 = lane & 15;
        const int mk = LENS ? live_blocks(m, b, gr.nl) : m;  // blocks k >= mk: no real key

        // scores and softmax over k for the query rows of this wave
        int lr[RT];
        float inv[RT], lse[RT];
        f32x4 sc[RT][NT];  // lane holds Z[k = 16t + 4g + qq][l] (log2 units) of row tile r
        RowFrags<T, D> bf[RT];
#pragma unroll
        for (int r = 0; r < RT; ++r) {
            lr[r] = (wave * RT + r) * 16 + c16;
#pragma unroll
            for (int c = 0; c < D / Mma<T>::KC; ++c)
                bf[r].f[c] = *reinterpret_cast<const typename Mma<T>::frag *>(Qs + lr[r] * LDQ + c * Mma<T>::KC +
                                                                              g * Mma<T>::KPL);
        }
#pragma unroll
        for (int t = 0; t < NT; ++t) {
            f32x4 acc[RT];
            gemm_scores_rt<T, D, RT>(APs + (16 * t + c16) * LDQ, bf, acc, g);
            const f32x4 bias = *reinterpret_cast<const f32x4 *>(cLs + 16 * t + 4 * g);
#pragma unroll
            for (int r = 0; r < RT; ++r) {
#pragma unroll
                for (int qq = 0; qq < 4; ++qq) sc[r][t][qq] = __builtin_fmaf(acc[r][qq], hd.s_log2e, -bias[qq]);
            }
        }
#pragma unroll
        for (int r = 0; r < RT; ++r) {
            const float mx = tiles_max<NT, RAGGED>(sc[r], mk, g);
            float sum = 0.f;
#pragma unroll
            for (int t = 0; t < NT; ++t) {
#pragma unroll
                for (int qq = 0; qq < 4; ++qq) {
                    float e = __builtin_amdgcn_exp2f(sc[r][t][qq] - mx);
                    if (RAGGED && 16 * t + 4 * g + qq >= mk) e = 0.f;
                    sum = (t == 0 && qq == 0) ? e : sum + e;
                    sc[r][t][qq] = e;
                }
            }
            sum = lanegroup_sum(sum);
            // tile rows l >= m carry no weight, nor does a head without a real key
            const bool live = lr[r] < m && (!LENS || mk > 0);
            inv[r] = live ? fast_rcp(sum) : 0.f;
            lse[r] = live ? row_lse(mx, sum) : 0.f;
        }
        float *objs = cLs + NM;  // one objective share per wave
        if (p.obj_part) {
            float part = 0.f;
#pragma unroll
            for (int r = 0; r < RT; ++r) part += lse[r];
            part = rows16_sum(part);
            if (lane == 0) objs[wave] = part;
        }
        __syncthreads();  // every wave is done reading alpha_L
        if (p.obj_part && tid == 0) {
            float f = 0.f;
            for (int w = 0; w < W; ++w) f += objs[w];
            p.obj_part[(bh * hd.T + hd.t - 1) * b + j] = f;
        }

        // P[l][k] = L[j][k][l] (row-major, k contiguous) into the alpha_L space
        T *Ps = APs;
#pragma unroll
        for (int r = 0; r < RT; ++r) {
#pragma unroll
            for (int t = 0; t < NT; ++t) {
                store4<T>(Ps + lr[r] * LDP + 16 * t + 4 * g, sc[r][t] * inv[r]);
            }
        }
        __syncthreads();

        // wave w: key-block columns k in tiles wave*RT + r
        int kr[RT];
        ProbFrags<T, NT> pf[RT];  // B operand: P[l-slots][k]
#pragma unroll
        for (int r = 0; r < RT; ++r) {
            kr[r] = (wave * RT + r) * 16 + c16;
            pf[r].gather(Ps, LDP, (wave * RT + r) * 16, lane);
            const f32x4 cs = gemm_colsum<T, NT>(pf[r]);  // c_R[k][j] = sum_l L[j][k][l]
            if (g == 0 && kr[r] < m) p.cR[bh * N + (int64_t)j * m + kr[r]] = cs[0];
        }
        f32x4 out[RT][D / 16];
#pragma unroll
        for (int vt = 0; vt < D / 16; ++vt) {
            f32x4 acc[RT];
            gemm_aggregate_rt<T, NT, RT>(Qs, LDQ, 16 * vt, pf, acc, lane);
#pragma unroll
            for (int r = 0; r < RT; ++r) out[r][vt] = acc[r];
        }
        const auto dd = head_dim<DK>(hd.d);  // states: rows of d elements
#pragma unroll
        for (int r = 0; r < RT; ++r)  // alpha_R[k][j] (k-major)
            store_row<T, D>(kr[r] < m ? p.aR + bh * N * dd + ((int64_t)kr[r] * b + j) * dd : nullptr, out[r],
                            1.0f, lane, dd);
    }
};

// ---------------------------------------------------------------------------------------
// Last L half-step fused with the second Monarch product and the store of O
// for (head bh, class j); each wave owns RT tiles of 16 query rows l.
// ---------------------------------------------------------------------------------------
template <typename T, int NM, int D, bool RAGGED, bool LENS = false> struct Apply {
    static_assert(!LENS || RAGGED, "per-sequence lengths need the masked softmax");
    static constexpr int NT = NM / 16, RT = Split<NT>::RT, W = Split<NT>::W, NTH = 64 * W;
    static constexpr bool NF = NormFirst<NT, D>::value;
    static constexpr int LDK = Ld<T, D>::row;
    static constexpr int LDS_BYTES = 2 * NM * LDK * (int)sizeof(T) + NM * 4 + W * 4;

    struct Regs {
        TileChunks<T, NM, D, NTH> at, yt;  // alpha_L[j], Y[j] (rows k)
        float cl;                          // c_L[k = tid][j]
        RowFrags<T, D> bf[RT];             // Qbar[j] rows l
        int nl;                            // real rows of the head (LENS)
    };

    template <int DK, bool RV>
    __device__ static void fetch(const Bufs<T> &p, const HeadDims &hd, int64_t bh, int j, int tid, Regs &gr)
    {
        const int m = hd.m, b = hd.b;
        const int64_t N = (int64_t)m * b;
        const int lane = tid & 63, wave = tid >> 6;
        const auto dd = head_dim<DK>(hd.d);
        const int64_t hoff = bh * N * dd;  // states: rows of d elements
        const T *al = p.aL + hoff + (int64_t)j * m * dd;
        const T *yj = p.Y + hoff + (int64_t)j * m * dd;
        gr.at.fetch([=](int kk) { return al + (int64_t)kk * dd; }, m, tid, dd);
        gr.yt.fetch([=](int kk) { return yj + (int64_t)kk * dd; }, m, tid, dd);
        const T *qb = p.q + bh * (int64_t)hd.n * dd + mrow_u<RV>(hd, j) * dd;  // Qbar[j][0]
        const int64_t sq = rstep<RV>(hd, b) * dd;
#pragma unroll
        for (int r = 0; r < RT; ++r) {
            const int l = (wave * RT + r) * 16 + (lane & 15);
            gr.bf[r].load((int64_t)l * b + j < hd.n ? qb + l * sq : nullptr, lane >> 4, dd);  // Qbar[j][l]; zero if padded
        }
        gr.cl = tid < m ? p.cL[bh * N + (int64_t)tid * b + j] : 0.f;
        if constexpr (LENS) gr.nl = live_rows(hd, bh);
    }

    __device__ static void stage(const HeadDims &, const Regs &gr, char *lds, int tid)
    {
        T *As = reinterpret_cast<T *>(lds);
        T *Ys = As + NM * LDK;
        gr.at.template stage<LDK>(As, tid);
        gr.yt.template stage<LDK>(Ys, tid);
        if (tid < NM) reinterpret_cast<float *>(Ys + NM * LDK)[tid] = gr.cl * kLog2e;
    }

    // After stage() and a barrier.
    template <int DK, bool RV>
    __device__ static void compute(const Bufs<T> &p, const HeadDims &hd, int64_t bh, int j, const Regs &gr,
                                   char *lds, int tid)
    {
        T *As = reinterpret_cast<T *>(lds);
        T *Ys = As + NM * LDK;
        float *cLs = reinterpret_cast<float *>(Ys + NM * LDK);
        const int m = hd.m, b = hd.b;
        const int lane = tid & 63, wave = tid >> 6;
        const int g = lane >> 4, c16 = lane & 15;
        const int nl = LENS ? gr.nl : hd.n;
        const int mk = LENS ? live_blocks(m, b, nl) : m;  // blocks k >= mk: no real key
        int lr[RT];
#pragma unroll
        for (int r = 0; r < RT; ++r) lr[r] = (wave * RT + r) * 16 + c16;
        RowFrags<T, D> bfq[RT];  // with per-sequence lengths: query rows beyond the length zeroed
        if constexpr (LENS) {
#pragma unroll
            for (int r = 0; r < RT; ++r) {
                bfq[r] = gr.bf[r];
                bfq[r].clear_if((int64_t)lr[r] * b + j >= nl);
            }
        }
        const RowFrags<T, D> *bf = LENS ? bfq : gr.bf;

        f32x4 sc[RT][NT];  // lane holds Z[k = 16t + 4g + qq][l] (log2 units) of row tile r
#pragma unroll
        for (int t = 0; t < NT; ++t) {
            f32x4 acc[RT];
            gemm_scores_rt<T, D, RT>(As + (16 * t + c16) * LDK, bf, acc, g);
            const f32x4 bias = *reinterpret_cast<const f32x4 *>(cLs + 16 * t + 4 * g);
#pragma unroll
            for (int r = 0; r < RT; ++r) {
#pragma unroll
                for (int qq = 0; qq < 4; ++qq) sc[r][t][qq] = __builtin_fmaf(acc[r][qq], hd.s_log2e, -bias[qq]);
            }
        }
        ProbFrags<T, NT> pf[RT];
        float inv[RT], lse[RT];
#pragma unroll
        for (int r = 0; r < RT; ++r) {
            const float mx = tiles_max<NT, RAGGED>(sc[r], mk, g);
            float sum = 0.f;
#pragma unroll
            for (int t = 0; t < NT; ++t) {
#pragma unroll
                for (int qq = 0; qq < 4; ++qq) {
                    float e = __builtin_amdgcn_exp2f(sc[r][t][qq] - mx);
                    if (RAGGED && 16 * t + 4 * g + qq >= mk) e = 0.f;
                    sum = (t == 0 && qq == 0) ? e : sum + e;
                    sc[r][t][qq] = e;
                }
            }
            sum = lanegroup_sum(sum);
            const bool any = !LENS || mk > 0;  // a head without a real key has L = 0
            inv[r] = any ? fast_rcp(sum) : 0.f;
            lse[r] = (lr[r] < m && any) ? row_lse(mx, sum) : 0.f;
            if constexpr (NF) {
#pragma unroll
                for (int t = 0; t < NT; ++t) sc[r][t] *= inv[r];
                inv[r] = 1.0f;
            }
            pf[r].pack(sc[r]);  // !NF: unnormalised, the row sum is divided out of O below
        }
        if (p.obj_part) {  // objective share of class j at the last step (uniform branch)
            float *objs = cLs + NM;
            float part = 0.f;
#pragma unroll
            for (int r = 0; r < RT; ++r) part += lse[r];
            part = rows16_sum(part);
            if (lane == 0) objs[wave] = part;
            __syncthreads();
            if (tid == 0) {
                float f = 0.f;
                for (int w = 0; w < W; ++w) f += objs[w];
                p.obj_part[(bh * hd.T + hd.t - 1) * b + j] = f;
            }
        }
        f32x4 o[RT][D / 16];
#pragma unroll
        for (int vt = 0; vt < D / 16; ++vt) {
            f32x4 acc[RT];
            gemm_aggregate_rt<T, NT, RT>(Ys, LDK, 16 * vt, pf, acc, lane);
#pragma unroll
            for (int r = 0; r < RT; ++r) o[r][vt] = acc[r];
        }
        const auto dd = head_dim<DK>(hd.d);
        T *ob = p.out + bh * (int64_t)hd.n * dd + mrow_u<RV>(hd, j) * dd;  // O[j], row 0 of class j
        const int64_t so = rstep<RV>(hd, b) * dd;
#pragma unroll
        for (int r = 0; r < RT; ++r) {  // rows nl..n-1 (batch padding) are written as zero
            const int64_t row = (int64_t)lr[r] * b + j;
            store_row<T, D>(row < hd.n ? ob + lr[r] * so : nullptr, o[r], (!LENS || row < nl) ? inv[r] : 0.f, lane,
                            dd);
        }
    }
};

// ---------------------------------------------------------------------------------------
// One launch per half-step.  The grid holds at most as many workgroups as
// are resident at once; workgroup i takes units i, i + gridDim.x, ... and
// issues the global loads of its next unit as soon as the current one is in
// LDS, so that they land while it computes.  `per` is the number of units
// per head (m for R, b for L).
// ---------------------------------------------------------------------------------------
template <typename U, int DK, bool RV, typename T>
__device__ inline void run_units_d(const Bufs<T> &p, const HeadDims &hd, int per, char *lds)
{
    const int tid = threadIdx.x;
    int64_t u = blockIdx.x;
    typename U::Regs cur, nxt;
    U::template fetch<DK, RV>(p, hd, u / per, (int)(u % per), tid, cur);
    while (true) {
        U::stage(hd, cur, lds, tid);
        __syncthreads();
        const int64_t un = u + gridDim.x;
        if (un < hd.units) U::template fetch<DK, RV>(p, hd, un / per, (int)(un % per), tid, nxt);
        U::template compute<DK, RV>(p, hd, u / per, (int)(u % per), cur, lds, tid);
        if (un >= hd.units) break;
        __syncthreads();  // LDS is restaged next
        cur = nxt;
        u = un;
    }
}

// The unit loop of the usual call (d fills the tile, no pre-padding), with
// the head dimension a constant and no row reversal, or of any other call
// (one uniform branch per workgroup; both loops are compiled into the kernel).
template <typename U, int D, typename T> __device__ inline void run_units(const Bufs<T> &p, const HeadDims &hd, int per, char *lds)
{
    if (hd.d == D && !hd.rev)
        run_units_d<U, D, false>(p, hd, per, lds);
    else
        run_units_d<U, 0, true>(p, hd, per, lds);
}

// The unit that a launch runs, whose NTH threads are its workgroup.
template <typename T, int NB, int D, bool FIRST, bool FINAL, bool RAGGED, bool LENS>
using RUnit = typename std::conditional<std::is_same<T, float>::value, RHalf32<NB, D, FIRST, FINAL, RAGGED, LENS>,
                                        RHalf<T, NB, D, FIRST, FINAL, RAGGED, LENS>>::type;
template <typename T, int NM, int D, bool RAGGED, bool LENS>
using LUnit = typename std::conditional<std::is_same<T, float>::value, LHalf32<NM, D, RAGGED, LENS>,
                                        LHalf<T, NM, D, RAGGED, LENS>>::type;
template <typename T, int NM, int D, bool RAGGED, bool LENS>
using ApplyUnit = typename std::conditional<std::is_same<T, float>::value, Apply32<NM, D, RAGGED, LENS>,
                                            Apply<T, NM, D, RAGGED, LENS>>::type;

template <typename T, int NB, int D, bool FIRST, bool FINAL, bool RAGGED, bool LENS>
__global__ __launch_bounds__((RUnit<T, NB, D, FIRST, FINAL, RAGGED, LENS>::NTH)) void r_half_step(Bufs<T> p, HeadDims hd)
{
    using U = RUnit<T, NB, D, FIRST, FINAL, RAGGED, LENS>;
    __shared__ __attribute__((aligned(16))) char lds[U::LDS_BYTES];
    run_units<U, D>(p, hd, hd.m, lds);
}

template <typename T, int NM, int D, bool RAGGED, bool LENS>
__global__ __launch_bounds__((LUnit<T, NM, D, RAGGED, LENS>::NTH)) void l_half_step(Bufs<T> p, HeadDims hd)
{
    using U = LUnit<T, NM, D, RAGGED, LENS>;
    __shared__ __attribute__((aligned(16))) char lds[U::LDS_BYTES];
    run_units<U, D>(p, hd, hd.b, lds);
}

template <typename T, int NM, int D, bool RAGGED, bool LENS>
__global__ __launch_bounds__((ApplyUnit<T, NM, D, RAGGED, LENS>::NTH)) void monarch_apply(Bufs<T> p, HeadDims hd)
{
    using U = ApplyUnit<T, NM, D, RAGGED, LENS>;
    __shared__ __attribute__((aligned(16))) char lds[U::LDS_BYTES];
    run_units<U, D>(p, hd, hd.b, lds);
}

// f(M^(t); Q, K) of every (head, step): the objective shares summed over the
// b classes, in class order.  One thread per (head, step).
static __global__ __launch_bounds__(256) void objective_sum(const float *part, float *obj, int64_t units, int b)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= units) return;
    float f = 0.f;
    for (int j = 0; j < b; ++j) f += part[i * b + j];
    obj[i] = f;
}

// ---------------------------------------------------------------------------------------
// Exact softmax attention O = softmax(s Q K^T) V with the logsumexp of every
// row (eq. softmax_attention): the quality reference the Monarch output is
// measured against, and the upper bound of the objective (sum of the row
// logsumexps).  One workgroup of 4 waves per 64 query rows; wave w owns 16
// query rows (the B operand of the scores, in registers) and keeps an online
// softmax (running max, sum and output) over tiles of 64 keys.  Scores are
// transposed as in the half-steps (keys on the MFMA row axis), so the
// probabilities feed the V product straight from registers; the key and value
// tiles of the next step are fetched into registers while the current one is
// computed.
// ---------------------------------------------------------------------------------------
template <typename T, int D> struct ExactAttn {
    static constexpr int KT = 64, NT = KT / 16, W = 4, NTH = 64 * W;
    static constexpr int LDK = Ld<T, D>::row;
    static constexpr int LDS_BYTES = 2 * KT * LDK * (int)sizeof(T);

    struct Tiles {
        TileChunks<T, KT, D, NTH> kt, vt;
    };

    __device__ static void fetch(const T *kh, const T *vh, int n, int d, int key0, int tid, Tiles &g)
    {
        const int valid = n - key0 < KT ? n - key0 : KT;
        g.kt.fetch([=](int r) { return kh + (int64_t)(key0 + r) * d; }, valid, tid, d);
        g.vt.fetch([=](int r) { return vh + (int64_t)(key0 + r) * d; }, valid, tid, d);
    }

    __device__ static void run(const Bufs<T> &p, float *lse_out, int n, int d, float s_log2e, char *lds)
    {
        T *Ks = reinterpret_cast<T *>(lds);
        T *Vs = Ks + KT * LDK;
        const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, g = lane >> 4, c16 = lane & 15;
        const int64_t qblocks = (n + 63) / 64;
        const int64_t bh = blockIdx.x / qblocks;
        const int row = (int)(blockIdx.x % qblocks) * 64 + wave * 16 + c16;  // this lane's query row
        const int64_t hoff = bh * (int64_t)n * d;
        const T *qh = p.q + hoff, *kh = p.k + hoff, *vh = p.v + hoff;

        RowFrags<T, D> bf;
        bf.load(row < n ? qh + (int64_t)row * d : nullptr, g, d);
        float mx = kMasked, sum = 0.f;  // running max (log2 units) and sum of this query row
        f32x4 o[D / 16];
#pragma unroll
        for (int vt = 0; vt < D / 16; ++vt) o[vt] = f32x4{0.f, 0.f, 0.f, 0.f};

        Tiles cur, nxt;
        fetch(kh, vh, n, d, 0, tid, cur);
        for (int key0 = 0; key0 < n; key0 += KT) {
            cur.kt.template stage<LDK>(Ks, tid);
            cur.vt.template stage<LDK>(Vs, tid);
            __syncthreads();
            if (key0 + KT < n) fetch(kh, vh, n, d, key0 + KT, tid, nxt);
            const int kv = n - key0;  // keys >= kv of this tile are beyond N
            f32x4 sc[NT];             // lane holds u = s log2(e) q.k for keys 16t + 4g + qq
#pragma unroll
            for (int t = 0; t < NT; ++t) {
                f32x4 acc;
                gemm_scores_rt<T, D, 1>(Ks + (16 * t + c16) * LDK, &bf, &acc, g);
                sc[t] = acc * s_log2e;
            }
            const float tmax = tiles_max<NT, true>(sc, kv, g);
            const float mnew = max_nan(mx, tmax);
            const float corr = __builtin_amdgcn_exp2f(mx - mnew);
            float tsum = 0.f;
#pragma unroll
            for (int t = 0; t < NT; ++t) {
#pragma unroll
                for (int qq = 0; qq < 4; ++qq) {
                    float e = __builtin_amdgcn_exp2f(sc[t][qq] - mnew);
                    if (16 * t + 4 * g + qq >= kv) e = 0.f;
                    tsum += e;
                    sc[t][qq] = e;
                }
            }
            sum = sum * corr + lanegroup_sum(tsum);
            mx = mnew;
            ProbFrags<T, NT> pf;
            pf.pack(sc);
#pragma unroll
            for (int vt = 0; vt < D / 16; ++vt) o[vt] = o[vt] * corr + gemm_aggregate<T, NT>(Vs, LDK, 16 * vt, pf, lane);
            __syncthreads();  // the tiles are restaged next
            cur = nxt;
        }
        const float inv = fast_rcp(sum);
        store_row<T, D>(row < n ? p.out + hoff + (int64_t)row * d : nullptr, o, inv, lane, d);
        if (lse_out && g == 0 && row < n) lse_out[bh * n + row] = row_lse(mx, sum);
    }
};

template <typename T, int D>
__global__ __launch_bounds__(256) void exact_attention(Bufs<T> p, float *lse, int n, int d, float s_log2e)
{
    using U = ExactAttn<T, D>;
    __shared__ __attribute__((aligned(16))) char lds[U::LDS_BYTES];
    U::run(p, lse, n, d, s_log2e, lds);
}

}  // namespace ma
