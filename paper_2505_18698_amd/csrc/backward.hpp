// Gradient of the MonarchAttention forward pass: reverse mode through the
// unrolled T steps of Sec. 3 (the paper gives no gradient; the sweep below is
// derived from the state form of its Implementation paragraph).
//
// Notation per head, with s = 1/sqrt(d), Qbar[j][l] = Q[l*b + j] (unscaled),
// Kbar[k][i] = K[k*b + i], and the states of step t as the forward stores
// them (alpha_R unscaled, the scale applied on the scores):
//   R update of block k:  Z_R[j][i] = s <alpha_R[k][j], Kbar[k][i]> / c_R[k][j]
//                         (keys i past the sequence masked), R = softmax_i Z_R,
//                         alpha_L[j][k] = sum_i R Kbar[k][i], c_L[j][k] = sum_i R log R,
//                         Y[j][k] = sum_i R Vbar[k][i] at the last step;
//   L update of class j:  Z_L[l][k] = s <Qbar[j][l], alpha_L[j][k]> - c_L[j][k],
//                         L = softmax_k Z_L, alpha_R'[k][j] = sum_l L Qbar[j][l],
//                         c_R'[k][j] = sum_l L (inputs of step t+1), and at the
//                         last step O[l*b + j] = sum_k L Y[j][k];
//   step 1 starts from L = I: alpha_R[k][j] = Q[k*b + j], c_R = 1.
// A softmax p = softmax(z) pulls dp back to dz = p (dp - <p, dp>).
//
// The sweep runs t = T .. 1, one launch per half-step:
//   l_bwd (class j of step t):  dL = dO . Y (t = T; also dY = L^T dO) or
//       dL = Qbar . d alpha_R' + d c_R' (t < T; also dQbar += L d alpha_R');
//       dW = s L (dL - <L, dL>) (the scale folded in);  dQbar += dW alpha_L,
//       d alpha_L = dW^T Qbar,  d c_L = -(1/s) sum_l dW.
//   r_bwd (block k of step t):  dR = d alpha_L . Kbar + d c_L (log R + 1)
//       (+ dY . Vbar at t = T, with dVbar = R^T dY);  dZ = R (dR - <R, dR>);
//       dKbar += R^T d alpha_L + (s dZ / c_R)^T alpha_R;
//       d alpha_R = (s dZ / c_R) Kbar;  d c_R = -sum_i dZ log R / c_R (the rows
//       of dZ sum to zero, so log R stands in for the logits);  at t = 1
//       d alpha_R is added to dQ (alpha_R = the rows of Q) and c_R is constant.
//
// Products.  The sweep's arithmetic is fp32: gradients, factors and
// accumulators are fp32, and a product runs on the bf16 matrix instruction
// over its operands' planes (planes.hpp, which states their range), 1 to 6
// instructions a tile and chunk.  An infinite dO gives infinities in dV, as
// fp32 products do; in the gradients of the factors they cancel to NaN.
//
// A unit (a block k of r_bwd, a class j of l_bwd) is one workgroup.  Its
// columns (keys i, or key blocks k) are shared out over the waves in groups of
// IPW 16-wide tiles, whose operands a wave holds in registers for the whole
// unit; its rows (j, or l) pass through LDS in chunks of C.  Per chunk:
//   1. the chunk's row operands go to LDS as planes (loaded a chunk ahead);
//   2. wave (jt, ig) forms the transposed score tiles of row tile jt and its
//      own columns, and the gradient of the factor, in the same registers
//      (lane: columns 16t + 4g + q of row lane % 16);
//   3. one exchange of partial row sums gives the softmax and its pull-back;
//   4. the factor and the gradient of its logits go to LDS as planes, and the
//      products that contract over the rows (into registers, for the whole
//      unit) and over the columns (a tile of the row operand's gradient) follow.
// A unit sizes its tiles by its own dimension (m for l_bwd, b for r_bwd).
//
// What bounds it: VALU issue and the latency of the phases between barriers.
// At 16 heads of 128 x 128 blocks, d = 64, T = 2, bf16, the four launches take
// r_bwd 194 and 120 us (t = 2, t = 1), l_bwd 145 and 160 us; on the fp32
// matrix instruction, with the factors in LDS as fp32, they took 390, 347,
// 289 and 345 us.  Their bytes alone (67 MB a state in fp32) take about 70 us
// each.  VALU is active 35% of the time (46% in r_bwd at t = 1), the matrix cores
// 23% in r_bwd, 13 and 17% in l_bwd.
//
// What it costs: one wave runs a 16-row unit that four waves ran on the fp32
// instruction, and where its rows are mostly padding its chain is longer.
// Gradients of blocks of one to three rows take 2 to 6% longer in fp32 and fp16,
// in fp32 at d > 96 up to 15% (91 heads of 2 x 1 rows, d = 128, T = 3: 64 -> 74 us;
// 281 of 12 x 2, d = 104: 202 -> 227).
//
// The gradients of the states and the dQ, dK accumulators are fp32 in the
// workspace.  Within a launch the units write disjoint rows, and launches that
// touch the same rows are ordered on the stream, so read-modify-writes need no
// atomics and the result is deterministic.  dq and dk are written in the
// element type by the step-1 R launch (the last one to touch them), dv by the
// step-T R launch.
#pragma once

#include "planes.hpp"

namespace ma {

template <typename T> struct BwdBufs {
    const T *q, *k, *v, *dout;  // [B*H][n][d]
    const T *aR, *aL, *Y;       // states of the step being undone ([m][b][d], [b][m][d], [b][m][d])
    const float *cR, *cL;       // c_R [b][m] (j-major), c_L [m][b] (k-major), as the forward writes them
    float *dQ, *dK;             // fp32 accumulators [B*H][n][d]
    T *dq, *dk, *dv;            // results [B*H][n][d]
    float *daL, *dcL, *dY;      // [b][m][D], [b][m], [b][m][D]: written by l_bwd, read by r_bwd of the step
    float *daR, *dcR;           // [m][b][D], [m][b]: written by r_bwd of step t, read by l_bwd of step t-1
};

struct BwdDims {
    int m, b, n, d;  // as in the forward (the states have rows of d elements, the fp32 state gradients of D)
    float s;         // 1/sqrt(d)
    // Per-sequence lengths (batch padding): head bh has lens[bh / H] real
    // rows, clamped to 0..n, or n when lens is null.  Rows past them count as
    // zero in the forward, so their gradients are zero.
    const int *lens = nullptr;
    int H = 1;
};

namespace bwd {

// Real rows of head bh (bh < 2^31: the grids are checked on the host).
__device__ inline int live_rows(const BwdDims &dm, int64_t bh)
{
    if (!dm.lens) return dm.n;
    const int len = dm.lens[(int)bh / dm.H];
    return len < 0 ? 0 : len > dm.n ? dm.n : len;
}

// The four columns 16t + 4g + q that a lane holds of row `row` of a factor, as
// three planes.
template <Reach R> __device__ inline void store_factor(__bf16 *row, int plane, f32x4 x)
{
    const float v[4] = {x[0], x[1], x[2], x[3]};
    bf16x4 p[3];
    split<3, 4, R>(v, p);
#pragma unroll
    for (int a = 0; a < 3; ++a) *reinterpret_cast<bf16x4 *>(row + a * plane) = p[a];
}

// Keeps the compiler from moving LDS reads above this point: hoisted, the
// operands of all products of a chunk would be live at once.
__device__ inline void reads_stay() { asm volatile("" ::: "memory"); }

// e^x (x <= 0) in natural units: the pull-backs keep their logits unscaled, so
// that the rounding of fp32 logits is not added to.
__device__ inline float exp_nat(float x) { return __builtin_amdgcn_exp2f(x * kLog2e); }

// 1 / x for x >= 1: the hardware reciprocal and one Newton step (to the last bit or so).
__device__ inline float rcp1(float x)
{
    const float r = fast_rcp(x);
    return __builtin_fmaf(__builtin_fmaf(-x, r, 1.f), r, r);
}

// The row statistics take the gradients times 2^-8: the sums of at most 128
// terms e g, with e <= 1 not yet divided by their sum, then stay finite
// wherever g is.  (Powers of two, so the bits are those without it.)
constexpr float kStat = 0.00390625f, kUnstat = 256.f;

// What the waves of a unit exchange about a row of a factor p = e^z / sum e^z
// and its gradient g: of this wave's columns, the maximum of z, the sum of
// e = e^(z - max), and the sum of e g.  The pull-back needs g - <p, g>, which
// cancels where one weight dominates: with fp32 elements (REF) a wave gives
// the mean of g under its own weights and the sum of e (g - mean) instead, so
// that the differences, and not the values, carry the rounding.
template <bool REF> struct RowStat {
    float mx, sum, dot, rest;
    float scale, mean, fix;  // of the whole row: p = e scale, g - <p, g> = (g - mean) - fix

    // from this lane's columns (the four lane groups of a row hold its wave's)
    template <int N> __device__ inline void own(float mx_, const f32x4 (&e)[N], const f32x4 (&g)[N])
    {
        mx = mx_;
        sum = dot = rest = 0.f;
#pragma unroll
        for (int t = 0; t < N; ++t) {
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                sum += e[t][q];
                dot = __builtin_fmaf(e[t][q], g[t][q], dot);
            }
        }
        sum = lanegroup_sum(sum);
        dot = lanegroup_sum(dot);
        if constexpr (REF) {
            dot = sum != 0.f ? dot * fast_rcp(sum) : 0.f;  // the mean; NaN stays
#pragma unroll
            for (int t = 0; t < N; ++t) {
#pragma unroll
                for (int q = 0; q < 4; ++q) rest = __builtin_fmaf(e[t][q], g[t][q] - dot, rest);
            }
            rest = lanegroup_sum(rest);
        }
    }

    // The row of which this is one of NIG parts (in LDS, `step` apart); g of a
    // part is g + slope * (its maximum - the row's).  !live: a row of zeros.
    template <int NIG> __device__ inline void whole(const f32x4 *parts, int step, float slope, bool live)
    {
        float M = mx, all = sum, acc = dot, left = rest;
        if constexpr (NIG > 1) {
            M = kMasked;
#pragma unroll
            for (int x = 0; x < NIG; ++x) M = max_nan(M, parts[x * step][0]);
            all = acc = left = 0.f;
#pragma unroll
            for (int x = 0; x < NIG; ++x) {
                const f32x4 o = parts[x * step];
                const float sh = o[1] != 0.f ? o[0] - M : 0.f;  // (NaN too) a part of masked columns only adds nothing
                const float f = o[1] != 0.f ? exp_nat(sh) : 0.f;
                all = __builtin_fmaf(f, o[1], all);
                if constexpr (REF)
                    acc = __builtin_fmaf(f * o[1], __builtin_fmaf(slope, sh, o[2]), acc);
                else
                    acc = __builtin_fmaf(f, __builtin_fmaf(slope * sh, o[1], o[2]), acc);
            }
        }
        const float inv = live ? rcp1(all) : 0.f;
        mean = (REF && NIG == 1) ? dot : live ? acc * inv : 0.f;
        if constexpr (REF) {
            if constexpr (NIG > 1) {
#pragma unroll
                for (int x = 0; x < NIG; ++x) {
                    const f32x4 o = parts[x * step];
                    const float sh = o[1] != 0.f ? o[0] - M : 0.f;
                    const float f = o[1] != 0.f ? exp_nat(sh) : 0.f;
                    left = __builtin_fmaf(f, __builtin_fmaf(o[1], __builtin_fmaf(slope, sh, o[2]) - mean, o[3]), left);
                }
            }
            fix = live ? left * inv : 0.f;
        } else {
            fix = 0.f;
        }
        mx = NIG > 1 ? mx - M : 0.f;  // this part's maximum less the row's
        scale = NIG > 1 ? exp_nat(mx) * inv : inv;
    }
    __device__ inline float centred(float g) const { return REF ? (g - mean) - fix : g - mean; }
};

// Sums over the 16 lanes of a row (DPP), every lane ending with the sum.
template <int CTRL> __device__ inline float dpp(float x)
{
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), CTRL, 0xf, 0xf, false));
}
__device__ inline float lanes16_sum(float x)
{
    x += dpp<0xB1>(x);   // quad: xor 1
    x += dpp<0x4E>(x);   // quad: xor 2
    x += dpp<0x141>(x);  // half row mirror
    return x + dpp<0x140>(x);  // row mirror
}

// ---------------------------------------------------------------------------------------
// Shape of a unit: S columns (the tile of b for r_bwd, of m for l_bwd), D the
// tile width, NP planes of the element type.
// ---------------------------------------------------------------------------------------
struct Plan {
    int C;      // rows of a chunk
    bool UL;    // the unit's main column operand (K, alpha_L) in LDS instead of registers
    bool XL;    // l_bwd, t < T: d alpha_R' in LDS instead of registers
    bool MUX;   // the two factors take turns in one LDS buffer
};

template <int S, int D, int NP, bool LK, bool LAST> struct Shape {
    // Two workgroups a compute unit (K in LDS, the factors in turn, 128 VGPRs)
    // where that needs no spills: r_bwd before the last step at 128 x 64, 126 us
    // a launch against 178 us with one.  The others at that size hold dY's or
    // d alpha_R's operands as well and spill at 128 VGPRs: r_bwd of the last
    // step took 288 us against 212 us with one workgroup, l_bwd 231 against 152.
    static constexpr bool TWO = S == 128 && D == 64 && NP == 1 && !LK && !LAST;
    static constexpr int IPW = S >= 64 ? 2 : 1, NIG = S / 16 / IPW;  // column tiles per wave, column groups
    static constexpr int KDI = S >= 32 ? 32 : 16, NKI = S / KDI;     // contraction over the columns
    static constexpr int LDX = D + 16, LDP = S + 8;  // LDS rows: operands, factors (bank conflicts: see Ld, LHalf)
    static constexpr int NC = D / 32, NDT = D / 16;
    // planes of the row operands (r: alpha_R, d alpha_L and dY; l: Q and dO)
    static constexpr int PR = LK ? NP * (LAST ? 2 : 1) : NP + 3 + (LAST ? 3 : 0);
    static constexpr int PX = LK && !LAST ? 3 : NP;  // planes of Y or d alpha_R'

    static constexpr int dt2(int) { return (NDT + NIG - 1) / NIG; }  // tiles of the row gradient per wave
    static constexpr int regs(Plan p)  // VGPRs that live through the unit
    {
        const int njt = p.C / 16, dh = njt;
        int r = IPW * (NDT / dh) * 4 * (LAST ? 2 : 1);               // accumulators
        if (!p.UL) r += (IPW * NC + dt2(0) * NKI) * NP * 4;           // K, alpha_L: rows and columns
        if (LK) {
            if (!p.XL) r += IPW * NC * PX * 4 + (LAST ? 0 : dt2(0) * NKI * 12);
            r += IPW * 12;
        } else if (LAST) {
            r += IPW * NC * NP * 4;  // V
        }
        return r;
    }
    static constexpr int unit_bytes(Plan p) { return ((p.UL ? NP : 0) + (p.XL ? 3 : 0)) * S * LDX * 2; }
    static constexpr int rows_bytes(Plan p) { return PR * p.C * LDX * 2; }
    static constexpr int fact_bytes(Plan p) { return (p.MUX ? 1 : 2) * 3 * p.C * LDP * 2; }
    static constexpr int stat_bytes(Plan p) { return NIG * p.C * 20 + p.C * 8 + (LK ? S * 8 : 0); }
    static constexpr int lds_bytes(Plan p)
    {
        // the column operands pass through LDS once on their way to registers
        const int all = unit_bytes(p) + rows_bytes(p) + fact_bytes(p) + stat_bytes(p);
        const int main = p.UL ? 0 : NP * S * LDX * 2;
        const int x = LK && !LAST && !p.XL ? unit_bytes(p) + 3 * S * LDX * 2 : 0;
        return all > main ? (all > x ? all : x) : (main > x ? main : x);
    }
    // The first plan that fits the LDS and keeps the unit's operands within 168
    // VGPRs (208 where none does): registers before LDS for the operands (no
    // reads in the chunk loop), both factors in LDS at once before in turn (two
    // barriers fewer a chunk), chunks of 32 rows before 16 (a full contraction).
    static constexpr Plan pick()
    {
        if (TWO) return Plan{32, true, false, true};
        const int cmax = S >= 32 ? 32 : 16;
        for (int most = 168; most <= 208; most += 40)
            for (int c = cmax; c >= 16; c /= 2)
                for (int o = 0; o < 4; ++o)
                    for (int x = 0; x < 2; ++x) {
                        const Plan p{c, (o & 2) != 0, (o & 1) != 0, x == 1};
                        if (p.XL && !(LK && !LAST)) continue;
                        if (regs(p) <= most && lds_bytes(p) <= 160 * 1024) return p;
                    }
        return Plan{0, false, false, false};
    }
    static constexpr Plan P = pick();
    static_assert(P.C > 0, "no plan fits a compute unit");
    static constexpr int C = P.C, NJT = C / 16, W = NJT * NIG, NTH = 64 * W, KDJ = C;
    static constexpr int DH = NJT, DTW = NDT / DH;  // head-dimension parts, tiles of one
    static constexpr int DT2 = dt2(0);
    static constexpr int PLU = S * LDX, PLR = C * LDX, PLP = C * LDP;  // plane strides
    static constexpr int LDS_BYTES = lds_bytes(P);
    // Waves a SIMD that the registers are held to, where it takes no spills (the
    // compiler otherwise ends one or two registers over the step).
    static constexpr int waves()
    {
        if (TWO) return 4;
        if (D == 64 && NP == 1 && LK && LAST && S <= 32) return S == 16 ? 3 : 4;
        if (D == 64 && NP == 1 && !LK && !LAST && S == 64) return 3;
        if (S == 16 && (D <= 96 || (NP == 1 && !LK && !LAST))) return 2;
        return 1;
    }
    static constexpr int WAVES = waves();
};

// Waves of a unit's workgroup (the launch bound).
template <typename T, int S, int D, bool LK, bool LAST> constexpr int unit_threads = Shape<S, D, planes_of<T>, LK, LAST>::NTH;

// ---------------------------------------------------------------------------------------
// The L update of class j of step t undone (LAST: t = T, the update that also
// produced O).  S >= m: columns k, rows l.
// ---------------------------------------------------------------------------------------
template <typename T, int S, int D, bool LAST, bool LENS = false> struct LBwd {
    static constexpr int NP = planes_of<T>;
    using H = Shape<S, D, NP, true, LAST>;
    static constexpr Plan P = H::P;
    static constexpr int IPW = H::IPW, NIG = H::NIG, C = H::C, NJT = H::NJT, NTH = H::NTH, LDX = H::LDX, LDP = H::LDP;
    static constexpr int PX = H::PX;
    using KI = Frag<H::KDI>;
    using KJ = Frag<H::KDJ>;

    __device__ static void run(const BwdBufs<T> &p, const BwdDims &dm, char *lds)
    {
        const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, g = lane >> 4, c16 = lane & 15;
        const int jt = wave % NJT, ig = wave / NJT;
        const int m = dm.m, b = dm.b, n = dm.n, d = dm.d;
        const int64_t bh = blockIdx.x / b;
        const int j = blockIdx.x % b;
        const int nl = LENS ? live_rows(dm, bh) : n;
        const int ml = (nl - j + b - 1) / b;                 // real rows l: l*b + j < nl
        const int mk = LENS ? min(m, (nl + b - 1) / b) : m;  // key blocks k < mk hold a real key
        const int64_t Np = (int64_t)m * b, toff = bh * n * d, soff = bh * Np * D, coff = bh * Np;
        const int64_t xoff = bh * Np * d;  // the forward's states: rows of d elements

        __bf16 *US = reinterpret_cast<__bf16 *>(lds);           // alpha_L[j] (UL)
        __bf16 *XS = US + (P.UL ? NP * H::PLU : 0);             // d alpha_R' (XL)
        __bf16 *Qs = XS + (P.XL ? 3 * H::PLU : 0);              // Qbar rows of the chunk
        __bf16 *Gs = Qs + NP * H::PLR;                          // dO rows (LAST)
        __bf16 *Ls = Gs + (LAST ? NP * H::PLR : 0);             // L
        __bf16 *Ws = P.MUX ? Ls : Ls + 3 * H::PLP;              // dW
        f32x4 *stat = reinterpret_cast<f32x4 *>(Ws + 3 * H::PLP);  // [NIG][C]
        float *sums = reinterpret_cast<float *>(stat + NIG * C);   // [NJT][S]

        // Qbar[j], dO of class j: rows step_l apart; rows k of alpha_L[j] and Y[j], d apart, or of d alpha_R'
        const int step_l = b * d;
        const T *qb = p.q + toff + (int64_t)j * d, *gb = p.dout + toff + (int64_t)j * d;
        const T *ab = p.aL + xoff + (int64_t)j * m * d, *yb = p.Y + xoff + (int64_t)j * m * d;
        const float *xb = p.daR + soff + (int64_t)j * D;
        float *dqb = p.dQ + toff + (int64_t)j * d;

        // the unit's column operands
        bf16x8 aF[P.UL ? 1 : IPW][P.UL ? 1 : H::NC][NP], xF[P.XL ? 1 : IPW][P.XL ? 1 : H::NC][PX];
        KI aT[P.UL ? 1 : H::DT2][P.UL ? 1 : H::NKI][NP];
        KI xT[LAST || P.XL ? 1 : H::DT2][LAST || P.XL ? 1 : H::NKI][3];
        Rows<T, NP, S, D, LDX, NTH> ua;
        ua.fetch(ab, d, m, d, tid);
        Rows<float, 3, S, D, LDX, NTH> ux;
        if constexpr (!LAST) ux.fetch(xb, b * D, m, d, tid);
        Rows<T, NP, C, D, LDX, NTH> qr;
        Rows<T, NP, C, D, LDX, NTH, Reach::kInf> gr;
        qr.fetch(qb, step_l, min(max(ml, 0), C), d, tid);
        if constexpr (LAST) gr.fetch(gb, step_l, min(max(ml, 0), C), d, tid);
        f32x4 cl[IPW], dcr[IPW];  // c_L[j][k], d c_R'[k][j] times kStat
#pragma unroll
        for (int t = 0; t < IPW; ++t) {
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int k = (ig * IPW + t) * 16 + 4 * g + q;
                cl[t][q] = Span(p.cL + coff + j).load1((uint32_t)(k * b) * 4, k < m);
                dcr[t][q] = 0.f;
                if constexpr (!LAST) dcr[t][q] = kStat * Span(p.dcR + coff + j).load1((uint32_t)(k * b) * 4, k < m);
            }
            const int k = (ig * IPW + t) * 16 + c16;
            if constexpr (LAST) {
#pragma unroll
                for (int c = 0; c < H::NC; ++c) load_chunk<T>(Span(yb), k, k < m, c, g, d, xF[t][c]);
            }
        }
        if constexpr (P.UL) {
            ua.stage(US, tid);
        } else {
            __bf16 *As = US;
            ua.stage(As, tid);
            __syncthreads();
#pragma unroll
            for (int t = 0; t < IPW; ++t) {
#pragma unroll
                for (int c = 0; c < H::NC; ++c) read_chunk<NP>(As + ((ig * IPW + t) * 16 + c16) * LDX, H::PLU, c, g, aF[t][c]);
            }
#pragma unroll
            for (int x = 0; x < H::DT2; ++x) {
                const int dt = min(ig + x * NIG, H::NDT - 1);
#pragma unroll
                for (int c = 0; c < H::NKI; ++c) read_cols<H::KDI, NP>(As, H::PLU, LDX, H::KDI * c, 16 * dt, lane, aT[x][c]);
            }
            __syncthreads();
        }
        if constexpr (!LAST) {
            if constexpr (P.XL) {
                ux.stage(XS, tid);
            } else {
                ux.stage(Qs, tid);
                __syncthreads();
#pragma unroll
                for (int t = 0; t < IPW; ++t) {
#pragma unroll
                    for (int c = 0; c < H::NC; ++c) read_chunk<3>(Qs + ((ig * IPW + t) * 16 + c16) * LDX, H::PLU, c, g, xF[t][c]);
                }
#pragma unroll
                for (int x = 0; x < H::DT2; ++x) {
                    const int dt = min(ig + x * NIG, H::NDT - 1);
#pragma unroll
                    for (int c = 0; c < H::NKI; ++c) read_cols<H::KDI, 3>(Qs, H::PLU, LDX, H::KDI * c, 16 * dt, lane, xT[x][c]);
                }
                __syncthreads();
            }
        }

        f32x4 daL[IPW][H::DTW], dY[LAST ? IPW : 1][LAST ? H::DTW : 1];  // d alpha_L^T, dY^T: sums over all rows l
        f32x4 dcl[IPW];                                                 // sums over this lane's rows of dW
#pragma unroll
        for (int t = 0; t < IPW; ++t) {
            dcl[t] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int x = 0; x < H::DTW; ++x) {
                daL[t][x] = f32x4{0.f, 0.f, 0.f, 0.f};
                if constexpr (LAST) dY[t][x] = f32x4{0.f, 0.f, 0.f, 0.f};
            }
        }

        for (int l0 = 0; l0 < m; l0 += C) {
            const int lc = min(max(ml - l0, 0), C);  // live rows of the chunk
            qr.stage(Qs, tid);
            if constexpr (LAST) gr.stage(Gs, tid);
            __syncthreads();
            // this lane's part of dQ's tiles, to be added to
            const int l = jt * 16 + c16;
            const Span dqs(dqb + (int64_t)l0 * step_l);
            f32x4 dqo[H::DT2];
            if constexpr (!LAST) {
#pragma unroll
                for (int x = 0; x < H::DT2; ++x) {
                    const int e = 16 * (ig + x * NIG) + 4 * g;
                    dqo[x] = dqs.loadf((l * step_l + e) * 4, l < lc && e < d);
                }
            }
            {  // past the last chunk: every load out of range, no traffic
                const int l1 = l0 + C, nn = min(max(ml - l1, 0), C);
                qr.fetch(qb + (int64_t)l1 * step_l, step_l, nn, d, tid);
                if constexpr (LAST) gr.fetch(gb + (int64_t)l1 * step_l, step_l, nn, d, tid);
            }

            // scores <alpha_L[k], Qbar[l]> and dL = Y . dO or d alpha_R' . Qbar (lane: k = 16t + 4g + q of row l)
            f32x4 z[IPW], w[IPW];
            Score<NP == 3> zs[IPW], ws[IPW];
#pragma unroll
            for (int c = 0; c < H::NC; ++c) {
                bf16x8 qf[NP], gf[NP];
                reads_stay();
                read_chunk<NP>(Qs + (jt * 16 + c16) * LDX, H::PLR, c, g, qf);
                if constexpr (LAST) read_chunk<NP>(Gs + (jt * 16 + c16) * LDX, H::PLR, c, g, gf);
#pragma unroll
                for (int t = 0; t < IPW; ++t) {
                    const int r = ((ig * IPW + t) * 16 + c16) * LDX;
                    if constexpr (P.UL) {
                        bf16x8 f[NP];
                        read_chunk<NP>(US + r, H::PLU, c, g, f);
                        zs[t].add(f, qf);
                    } else {
                        zs[t].add(aF[t][c], qf);
                    }
                    if constexpr (LAST) {
                        ws[t].add(xF[t][c], gf);
                    } else if constexpr (P.XL) {
                        bf16x8 f[3];
                        read_chunk<3>(XS + r, H::PLU, c, g, f);
                        ws[t].add(f, qf);
                    } else {
                        ws[t].add(xF[t][c], qf);
                    }
                }
            }
#pragma unroll
            for (int t = 0; t < IPW; ++t) z[t] = zs[t].value(), w[t] = ws[t].value();
            // L = softmax_k(s score - c_L) and its pull-back
            float mx = kMasked;
#pragma unroll
            for (int t = 0; t < IPW; ++t) {
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    z[t][q] = __builtin_fmaf(z[t][q], dm.s, -cl[t][q]);
                    w[t][q] = __builtin_fmaf(w[t][q], kStat, dcr[t][q]);
                    if ((ig * IPW + t) * 16 + 4 * g + q < mk) mx = max_nan(mx, z[t][q]);
                }
            }
            mx = wave_xor_max<32>(wave_xor_max<16>(mx));
#pragma unroll
            for (int t = 0; t < IPW; ++t) {
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    z[t][q] = (ig * IPW + t) * 16 + 4 * g + q < mk ? exp_nat(z[t][q] - mx) : 0.f;
            }
            RowStat<NP == 3> st;
            st.own(mx, z, w);
            const bool live = l0 + jt * 16 + c16 < m && (!LENS || mk > 0);  // rows past m, no real key: L = 0
            if constexpr (NIG > 1) {
                if (g == 0) stat[ig * C + jt * 16 + c16] = f32x4{st.mx, st.sum, st.dot, st.rest};
                __syncthreads();
            }
            st.template whole<NIG>(stat + jt * 16 + c16, C, 0.f, live);
            const float us = dm.s * kUnstat;
            __bf16 *lrow = Ls + (jt * 16 + c16) * LDP, *wrow = Ws + (jt * 16 + c16) * LDP;
#pragma unroll
            for (int t = 0; t < IPW; ++t) {
                const int k = (ig * IPW + t) * 16 + 4 * g;
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    z[t][q] *= st.scale;                                  // L
                    w[t][q] = us * z[t][q] * st.centred(w[t][q]);  // dW
                }
                dcl[t] += w[t];
                store_factor<Reach::kUnit>(lrow + k, H::PLP, z[t]);
                if constexpr (!P.MUX) store_factor<Reach::kFinite>(wrow + k, H::PLP, w[t]);
            }
            __syncthreads();

            f32x4 dq[H::DT2];  // dQbar^T tiles (dt, jt)
#pragma unroll
            for (int x = 0; x < H::DT2; ++x) dq[x] = f32x4{0.f, 0.f, 0.f, 0.f};
            if constexpr (LAST) {
                // dY[k] += sum_l L[l][k] dO[l]
                KJ lf[IPW][3];
#pragma unroll
                for (int t = 0; t < IPW; ++t) read_cols<H::KDJ, 3>(Ls, H::PLP, LDP, 0, (ig * IPW + t) * 16, lane, lf[t]);
#pragma unroll
                for (int x = 0; x < H::DTW; ++x) {
                    KJ f[NP];
                    reads_stay();
                    read_cols<H::KDJ, NP>(Gs, H::PLR, LDX, 0, (jt * H::DTW + x) * 16, lane, f);
#pragma unroll
                    for (int t = 0; t < IPW; ++t) mma_planes_inf(f, lf[t], dY[t][x]);
                }
            } else {
                // dQbar[l] += sum_k L[l][k] d alpha_R'[k]
#pragma unroll
                for (int c = 0; c < H::NKI; ++c) {
                    KI r[3];
                    reads_stay();
                    read_row<H::KDI, 3>(lrow, H::PLP, H::KDI * c, g, r);
#pragma unroll
                    for (int x = 0; x < H::DT2; ++x) {
                        if (H::DT2 * NIG > H::NDT && ig + x * NIG >= H::NDT) continue;
                        if constexpr (P.XL) {
                            KI f[3];
                            read_cols<H::KDI, 3>(XS, H::PLU, LDX, H::KDI * c, 16 * min(ig + x * NIG, H::NDT - 1), lane, f);
                            mma_planes(f, r, dq[x]);
                        } else {
                            mma_planes(xT[x][c], r, dq[x]);
                        }
                    }
                }
            }
            if constexpr (P.MUX) {
                __syncthreads();
#pragma unroll
                for (int t = 0; t < IPW; ++t) store_factor<Reach::kFinite>(wrow + (ig * IPW + t) * 16 + 4 * g, H::PLP, w[t]);
                __syncthreads();
            }
            // d alpha_L[k] += sum_l dW[l][k] Qbar[l]
            {
                KJ wf[IPW][3];
#pragma unroll
                for (int t = 0; t < IPW; ++t) read_cols<H::KDJ, 3>(Ws, H::PLP, LDP, 0, (ig * IPW + t) * 16, lane, wf[t]);
#pragma unroll
                for (int x = 0; x < H::DTW; ++x) {
                    KJ f[NP];
                    reads_stay();
                    read_cols<H::KDJ, NP>(Qs, H::PLR, LDX, 0, (jt * H::DTW + x) * 16, lane, f);
#pragma unroll
                    for (int t = 0; t < IPW; ++t) mma_planes(f, wf[t], daL[t][x]);
                }
            }
            // dQbar[l] += sum_k dW[l][k] alpha_L[k]
#pragma unroll
            for (int c = 0; c < H::NKI; ++c) {
                KI r[3];
                reads_stay();
                read_row<H::KDI, 3>(wrow, H::PLP, H::KDI * c, g, r);
#pragma unroll
                for (int x = 0; x < H::DT2; ++x) {
                    if (H::DT2 * NIG > H::NDT && ig + x * NIG >= H::NDT) continue;
                    if constexpr (P.UL) {
                        KI f[NP];
                        read_cols<H::KDI, NP>(US, H::PLU, LDX, H::KDI * c, 16 * min(ig + x * NIG, H::NDT - 1), lane, f);
                        mma_planes(f, r, dq[x]);
                    } else {
                        mma_planes(aT[x][c], r, dq[x]);
                    }
                }
            }
#pragma unroll
            for (int x = 0; x < H::DT2; ++x) {
                const int e = 16 * (ig + x * NIG) + 4 * g;  // (tiles past the last have e >= D >= d)
                f32x4 v = dq[x];
                if constexpr (!LAST) v += dqo[x];
                dqs.template store<float>(v, (l * step_l + e) * 4, l < lc && e < d);
            }
            __syncthreads();  // the next chunk overwrites the rows and factors
        }

#pragma unroll
        for (int t = 0; t < IPW; ++t) {
            const int k = (ig * IPW + t) * 16 + c16;
#pragma unroll
            for (int x = 0; x < H::DTW; ++x) {
                const int e = (jt * H::DTW + x) * 16 + 4 * g;
                const int64_t u = soff + (int64_t)j * m * D;
                const uint32_t o = (k * D + e) * 4;
                Span(p.daL + u).store<float>(daL[t][x], o, k < m && e < d);
                if constexpr (LAST) Span(p.dY + u).store<float>(dY[t][x], o, k < m && e < d);
            }
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const float v = lanes16_sum(dcl[t][q]);
                if (c16 == 0) sums[jt * S + (ig * IPW + t) * 16 + 4 * g + q] = v;
            }
        }
        __syncthreads();
        for (int k = tid; k < m; k += NTH) {
            float v = sums[k];
            if constexpr (NJT > 1) v += sums[S + k];
            p.dcL[coff + (int64_t)j * m + k] = -v / dm.s;
        }
    }
};

// ---------------------------------------------------------------------------------------
// The R update of block k of step t undone (FIRST: t = 1, LAST: t = T).
// S >= b: columns i (keys), rows j.
// ---------------------------------------------------------------------------------------
template <typename T, int S, int D, bool FIRST, bool LAST, bool LENS = false> struct RBwd {
    static constexpr int NP = planes_of<T>;
    using H = Shape<S, D, NP, false, LAST>;
    static constexpr Plan P = H::P;
    static constexpr int IPW = H::IPW, NIG = H::NIG, C = H::C, NJT = H::NJT, NTH = H::NTH, LDX = H::LDX, LDP = H::LDP;
    using KI = Frag<H::KDI>;
    using KJ = Frag<H::KDJ>;

    __device__ static void run(const BwdBufs<T> &p, const BwdDims &dm, char *lds)
    {
        const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, g = lane >> 4, c16 = lane & 15;
        const int jt = wave % NJT, ig = wave / NJT;
        const int m = dm.m, b = dm.b, n = dm.n, d = dm.d;
        const int64_t bh = blockIdx.x / m;
        const int k = blockIdx.x % m;
        const int kn = min(b, n - k * b);                              // rows of block k in memory
        const int kv = LENS ? min(b, live_rows(dm, bh) - k * b) : kn;  // real keys (and query rows); <= 0: none
        const int64_t Np = (int64_t)m * b, toff = bh * n * d, soff = bh * Np * D, coff = bh * Np;
        const int64_t xoff = bh * Np * d;     // the forward's states: rows of d elements
        const int64_t row0 = (int64_t)k * b;  // first row of block k

        __bf16 *US = reinterpret_cast<__bf16 *>(lds);           // Kbar[k] (UL)
        __bf16 *As = US + (P.UL ? NP * H::PLU : 0);             // alpha_R rows of the chunk (Q at t = 1)
        __bf16 *Ds = As + NP * H::PLR;                          // d alpha_L rows
        __bf16 *Ys = Ds + 3 * H::PLR;                           // dY rows (LAST)
        __bf16 *Rs = Ys + (LAST ? 3 * H::PLR : 0);              // R
        __bf16 *Zs = P.MUX ? Rs : Rs + 3 * H::PLP;              // dZ s / c_R
        f32x4 *stat = reinterpret_cast<f32x4 *>(Zs + 3 * H::PLP);  // [NIG][C]
        float *part = reinterpret_cast<float *>(stat + NIG * C);   // [NIG][C]
        float *cRs = part + NIG * C, *dcLs = cRs + C;              // c_R, d c_L of the chunk's rows

        // rows j of alpha_R[k] (Q at t = 1), d apart; of d alpha_L and dY, step_j apart
        const int step_j = m * D;
        const T *ab = FIRST ? p.q + toff + row0 * d : p.aR + xoff + row0 * d;
        const T *kb = p.k + toff + row0 * d, *vb = p.v + toff + row0 * d;
        const float *db = p.daL + soff + (int64_t)k * D, *yb = p.dY + soff + (int64_t)k * D;
        const int na = FIRST ? kv : b;  // rows of alpha_R

        // the unit's column operands
        bf16x8 kF[P.UL ? 1 : IPW][P.UL ? 1 : H::NC][NP], vF[LAST ? IPW : 1][LAST ? H::NC : 1][NP];
        KI kT[P.UL ? 1 : H::DT2][P.UL ? 1 : H::NKI][NP];
        Rows<T, NP, S, D, LDX, NTH> uk;
        uk.fetch(kb, d, max(kv, 0), d, tid);
        Rows<T, NP, C, D, LDX, NTH> ar;
        Rows<float, 3, C, D, LDX, NTH> dr;
        Rows<float, 3, C, D, LDX, NTH, Reach::kInf> yr;
        float crr = 1.f, dclr = 0.f;
        auto fetch = [&](int j0) {
            const int jb = min(b - j0, C);
            ar.fetch(ab + (int64_t)j0 * d, d, min(max(na - j0, 0), C), d, tid);
            dr.fetch(db + (int64_t)j0 * step_j, step_j, jb, d, tid);
            if constexpr (LAST) yr.fetch(yb + (int64_t)j0 * step_j, step_j, jb, d, tid);
            const int64_t u = coff + (int64_t)j0 * m + k;
            crr = 1.f;
            if constexpr (!FIRST) {
                crr = Span(p.cR + u).load1((uint32_t)(tid * m) * 4, tid < jb);
                if (tid >= jb) crr = 1.f;
            }
            dclr = Span(p.dcL + u).load1((uint32_t)(tid * m) * 4, tid < jb);
        };
        fetch(0);
        if constexpr (LAST) {
#pragma unroll
            for (int t = 0; t < IPW; ++t) {
                const int i = (ig * IPW + t) * 16 + c16;
#pragma unroll
                for (int c = 0; c < H::NC; ++c)
                    load_chunk<T>(Span(vb), i, i < kv, c, g, d, vF[t][c]);
            }
        }
        if constexpr (P.UL) {
            uk.stage(US, tid);
        } else {
            uk.stage(As, tid);
            __syncthreads();
#pragma unroll
            for (int t = 0; t < IPW; ++t) {
#pragma unroll
                for (int c = 0; c < H::NC; ++c) read_chunk<NP>(As + ((ig * IPW + t) * 16 + c16) * LDX, H::PLU, c, g, kF[t][c]);
            }
#pragma unroll
            for (int x = 0; x < H::DT2; ++x) {
                const int dt = min(ig + x * NIG, H::NDT - 1);
#pragma unroll
                for (int c = 0; c < H::NKI; ++c) read_cols<H::KDI, NP>(As, H::PLU, LDX, H::KDI * c, 16 * dt, lane, kT[x][c]);
            }
            __syncthreads();
        }

        f32x4 dK[IPW][H::DTW], dV[LAST ? IPW : 1][LAST ? H::DTW : 1];  // dKbar^T, dVbar^T: sums over all rows j
#pragma unroll
        for (int t = 0; t < IPW; ++t) {
#pragma unroll
            for (int x = 0; x < H::DTW; ++x) {
                dK[t][x] = f32x4{0.f, 0.f, 0.f, 0.f};
                if constexpr (LAST) dV[t][x] = f32x4{0.f, 0.f, 0.f, 0.f};
            }
        }

        for (int j0 = 0; j0 < b; j0 += C) {
            const int jb = min(b - j0, C);                   // rows of the chunk
            const int jq = min(max(kv - j0, 0), C);          // rows of Q (t = 1)
            const int jn = min(max(kn - j0, 0), C);          // rows of dq in memory (t = 1)
            ar.stage(As, tid);
            dr.stage(Ds, tid);
            if constexpr (LAST) yr.stage(Ys, tid);
            if (tid < C) cRs[tid] = crr, dcLs[tid] = dclr;
            __syncthreads();
            const int jj = jt * 16 + c16;
            f32x4 dqo[FIRST ? H::DT2 : 1];  // this lane's part of dQ's tiles (t = 1)
            if constexpr (FIRST) {
                const Span s(p.dQ + toff + (row0 + j0) * d);
#pragma unroll
                for (int x = 0; x < H::DT2; ++x) {
                    const int e = 16 * (ig + x * NIG) + 4 * g;
                    dqo[x] = s.loadf((jj * d + e) * 4, jj < jq && e < d);
                }
            }
            fetch(j0 + C);  // past the last chunk: every load out of range, no traffic

            // scores <Kbar[i], alpha_R[j]> and dR = Kbar . d alpha_L (+ Vbar . dY) (lane: i = 16t + 4g + q of row j)
            f32x4 z[IPW], w[IPW];
            Score<NP == 3> zs[IPW], ws[IPW];
#pragma unroll
            for (int c = 0; c < H::NC; ++c) {
                const int r = (jt * 16 + c16) * LDX;
                bf16x8 af[NP], df[3];
                reads_stay();
                read_chunk<NP>(As + r, H::PLR, c, g, af);
                read_chunk<3>(Ds + r, H::PLR, c, g, df);
#pragma unroll
                for (int t = 0; t < IPW; ++t) {
                    if constexpr (P.UL) {
                        bf16x8 f[NP];
                        read_chunk<NP>(US + ((ig * IPW + t) * 16 + c16) * LDX, H::PLU, c, g, f);
                        zs[t].add(f, af);
                        ws[t].add(f, df);
                    } else {
                        zs[t].add(kF[t][c], af);
                        ws[t].add(kF[t][c], df);
                    }
                }
                if constexpr (LAST) {
                    reads_stay();
                    read_chunk<3>(Ys + r, H::PLR, c, g, df);
#pragma unroll
                    for (int t = 0; t < IPW; ++t) ws[t].add(vF[t][c], df);
                }
            }
#pragma unroll
            for (int t = 0; t < IPW; ++t) z[t] = zs[t].value(), w[t] = ws[t].value();
            // R = softmax_i and its pull-back.  The gradient of row j's logits needs d R + d c_L (log R + 1) up to
            // a constant of the row: d c_L times the logits less their maximum stands in for the second term.
            const bool live = jj < jb && (!LENS || kv > 0);  // a block of padding only has R = 0
            const float cr = cRs[jj], dcl = dcLs[jj] * kStat;
            const float sc = live ? dm.s / cr : 0.f;
            float mx = kMasked;
#pragma unroll
            for (int t = 0; t < IPW; ++t) {
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    if ((ig * IPW + t) * 16 + 4 * g + q < kv) mx = max_nan(mx, z[t][q]);
                }
            }
            // a wave of masked keys only: logits of zero here (their e is zero), no part in the row's maximum
            const bool none = ig * IPW * 16 >= kv;
            mx = none ? 0.f : wave_xor_max<32>(wave_xor_max<16>(mx)) * sc;
            f32x4 e4[IPW];
#pragma unroll
            for (int t = 0; t < IPW; ++t) {
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const float u = __builtin_fmaf(z[t][q], sc, -mx);
                    e4[t][q] = (ig * IPW + t) * 16 + 4 * g + q < kv ? exp_nat(u) : 0.f;
                    z[t][q] = u;
                    w[t][q] = __builtin_fmaf(dcl, u, w[t][q] * kStat);
                }
            }
            RowStat<NP == 3> st;
            st.own(mx, e4, w);
            if constexpr (NIG > 1) {
                if (g == 0) stat[ig * C + jj] = f32x4{none ? kMasked : st.mx, st.sum, st.dot, st.rest};
                __syncthreads();
            }
            st.template whole<NIG>(stat + jj, C, dcl, live);
            if (none) st.mx = st.scale = 0.f;
            const float off = dcl * st.mx, us = st.scale * kUnstat;
            __bf16 *rrow = Rs + jj * LDP, *zrow = Zs + jj * LDP;
            float dzlog = 0.f;
#pragma unroll
            for (int t = 0; t < IPW; ++t) {
                const int i = (ig * IPW + t) * 16 + 4 * g;
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const float r = e4[t][q] * st.scale;  // masked keys: 0
                    const float dz = (e4[t][q] * us) * st.centred(w[t][q] + off);
                    dzlog = __builtin_fmaf(dz, z[t][q] + st.mx, dzlog);
                    z[t][q] = r;
                    w[t][q] = dz * sc;
                }
                store_factor<Reach::kUnit>(rrow + i, H::PLP, z[t]);
                if constexpr (!P.MUX) store_factor<Reach::kFinite>(zrow + i, H::PLP, w[t]);
            }
            if constexpr (!FIRST) {
                dzlog = lanegroup_sum(dzlog);
                if (g == 0) part[ig * C + jj] = dzlog;
            }
            __syncthreads();
            if constexpr (!FIRST) {  // zero for a block of padding only (read by l_bwd)
                if (tid < jb) {
                    float v = 0.f;
#pragma unroll
                    for (int x = 0; x < NIG; ++x) v += part[x * C + tid];
                    p.dcR[coff + row0 + j0 + tid] = (!LENS || kv > 0) ? -v / cRs[tid] : 0.f;
                }
            }

            // dKbar[i] += sum_j R[j][i] d alpha_L[j];  dVbar[i] += sum_j R[j][i] dY[j]
            {
                KJ rf[IPW][3];
#pragma unroll
                for (int t = 0; t < IPW; ++t) read_cols<H::KDJ, 3>(Rs, H::PLP, LDP, 0, (ig * IPW + t) * 16, lane, rf[t]);
#pragma unroll
                for (int x = 0; x < H::DTW; ++x) {
                    KJ f[3];
                    reads_stay();
                    read_cols<H::KDJ, 3>(Ds, H::PLR, LDX, 0, (jt * H::DTW + x) * 16, lane, f);
#pragma unroll
                    for (int t = 0; t < IPW; ++t) mma_planes(f, rf[t], dK[t][x]);
                    if constexpr (LAST) {
                        reads_stay();
                        read_cols<H::KDJ, 3>(Ys, H::PLR, LDX, 0, (jt * H::DTW + x) * 16, lane, f);
#pragma unroll
                        for (int t = 0; t < IPW; ++t) mma_planes(f, rf[t], dV[t][x]);
                    }
                }
            }
            if constexpr (P.MUX) {
                __syncthreads();
#pragma unroll
                for (int t = 0; t < IPW; ++t) store_factor<Reach::kFinite>(zrow + (ig * IPW + t) * 16 + 4 * g, H::PLP, w[t]);
                __syncthreads();
            }
            // dKbar[i] += sum_j dZs[j][i] alpha_R[j]
            {
                KJ zf[IPW][3];
#pragma unroll
                for (int t = 0; t < IPW; ++t) read_cols<H::KDJ, 3>(Zs, H::PLP, LDP, 0, (ig * IPW + t) * 16, lane, zf[t]);
#pragma unroll
                for (int x = 0; x < H::DTW; ++x) {
                    KJ f[NP];
                    reads_stay();
                    read_cols<H::KDJ, NP>(As, H::PLR, LDX, 0, (jt * H::DTW + x) * 16, lane, f);
#pragma unroll
                    for (int t = 0; t < IPW; ++t) mma_planes(f, zf[t], dK[t][x]);
                }
            }
            // d alpha_R[j] = sum_i dZs[j][i] Kbar[i]: to the workspace, or at step 1 into dq
            f32x4 da[H::DT2];
#pragma unroll
            for (int x = 0; x < H::DT2; ++x) da[x] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int c = 0; c < H::NKI; ++c) {
                KI r[3];
                reads_stay();
                read_row<H::KDI, 3>(zrow, H::PLP, H::KDI * c, g, r);
#pragma unroll
                for (int x = 0; x < H::DT2; ++x) {
                    if (H::DT2 * NIG > H::NDT && ig + x * NIG >= H::NDT) continue;
                    if constexpr (P.UL) {
                        KI f[NP];
                        read_cols<H::KDI, NP>(US, H::PLU, LDX, H::KDI * c, 16 * min(ig + x * NIG, H::NDT - 1), lane, f);
                        mma_planes(f, r, da[x]);
                    } else {
                        mma_planes(kT[x][c], r, da[x]);
                    }
                }
            }
#pragma unroll
            for (int x = 0; x < H::DT2; ++x) {
                const int e = 16 * (ig + x * NIG) + 4 * g;
                if constexpr (FIRST) {  // rows past the length: zero
                    const f32x4 v = (!LENS || jj < jq) ? dqo[x] + da[x] : f32x4{0.f, 0.f, 0.f, 0.f};
                    Span(p.dq + toff + (row0 + j0) * d).store<T>(v, (jj * d + e) * (int)sizeof(T), jj < (LENS ? jn : jq) && e < d);
                } else {
                    Span(p.daR + soff + (row0 + j0) * D).store<float>(da[x], (jj * D + e) * 4, jj < jb && e < d);
                }
            }
            __syncthreads();  // the next chunk overwrites the rows and factors
        }

#pragma unroll
        for (int t = 0; t < IPW; ++t) {
            const int i = (ig * IPW + t) * 16 + c16;
#pragma unroll
            for (int x = 0; x < H::DTW; ++x) {
                const int e = (jt * H::DTW + x) * 16 + 4 * g;
                const int64_t u = toff + row0 * d;
                const uint32_t o = i * d + e;
                const bool in = i < (LENS && FIRST ? kn : kv) && e < d;  // at t = 1 rows past the length get zero
                f32x4 v = dK[t][x];
                if constexpr (!LAST) v += Span(p.dK + u).loadf(o * 4, i < kv && e < d);
                if (LENS && i >= kv) v = f32x4{0.f, 0.f, 0.f, 0.f};
                if constexpr (FIRST)
                    Span(p.dk + u).store<T>(v, o * (uint32_t)sizeof(T), in);
                else
                    Span(p.dK + u).store<float>(v, o * 4, in);
                if constexpr (LAST) {
                    if (LENS && i >= kv) dV[t][x] = f32x4{0.f, 0.f, 0.f, 0.f};
                    Span(p.dv + u).store<T>(dV[t][x], o * (uint32_t)sizeof(T), i < (LENS ? kn : kv) && e < d);
                }
            }
        }
    }
};

template <typename T, int S, int D, bool LAST, bool LENS>
__global__ __launch_bounds__((unit_threads<T, S, D, true, LAST>), (Shape<S, D, planes_of<T>, true, LAST>::WAVES)) void l_bwd(BwdBufs<T> p, BwdDims dm)
{
    using U = LBwd<T, S, D, LAST, LENS>;
    __shared__ __attribute__((aligned(16))) char lds[U::H::LDS_BYTES];
    U::run(p, dm, lds);
}

template <typename T, int S, int D, bool FIRST, bool LAST, bool LENS>
__global__ __launch_bounds__((unit_threads<T, S, D, false, LAST>), (Shape<S, D, planes_of<T>, false, LAST>::WAVES)) void r_bwd(BwdBufs<T> p, BwdDims dm)
{
    using U = RBwd<T, S, D, FIRST, LAST, LENS>;
    __shared__ __attribute__((aligned(16))) char lds[U::H::LDS_BYTES];
    U::run(p, dm, lds);
}

}  // namespace bwd
}  // namespace ma
