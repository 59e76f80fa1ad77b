// Host-side pieces shared by the C ABI (monarch_attn.hip) and the per-dtype
// dispatch units (dispatch_*.hip).
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

#include "../../include/monarch_attn.h"

namespace ma_host {

// Record a failure for monarch_attn_last_error() and return `code`.
int fail(int code, const char *fmt, ...) __attribute__((format(printf, 2, 3)));

inline int pad16(int64_t x) { return (int)((x + 15) / 16 * 16); }

// Tile size (16, 32, 64 or 128 rows) the kernels use for a block of n <= 128 rows.
inline int tile_rows(int64_t n)
{
    const int p = pad16(n);
    return p <= 16 ? 16 : p <= 32 ? 32 : p <= 64 ? 64 : 128;
}

// Kernel kinds reported by the timing interface.
enum Kind { kR = 0, kL = 1, kRFinal = 2, kApply = 3, kFused = 4, kObjSum = 5, kExact = 6, kBwdL = 7, kBwdR = 8,
            kGroup = 9 };

// Per-launch HIP events around every kernel when timing is enabled.
constexpr int kMaxLaunches = 2 * 64 + 2;
struct Timing {
    bool enabled = false;
    bool ready = false;
    int nlaunch = 0;
    int kind[kMaxLaunches];
    hipEvent_t ev[2 * kMaxLaunches];
    bool created = false;
};
extern Timing g_timing;

template <typename F> int launched(F &&f)
{
    f();
    return MA_OK;
}

struct Launcher {
    hipStream_t stream;
    bool timed;
    int n = 0;

    template <typename F> int run(int kind, F &&launch)
    {
        if (timed) {
            if (n >= kMaxLaunches) return fail(MA_EHIP, "too many launches to time");
            if (hipEventRecord(g_timing.ev[2 * n], stream) != hipSuccess) return fail(MA_EHIP, "hipEventRecord failed");
        }
        const int rc = launch();
        if (rc != MA_OK) return rc;
        if (timed) {
            g_timing.kind[n] = kind;
            if (hipEventRecord(g_timing.ev[2 * n + 1], stream) != hipSuccess) return fail(MA_EHIP, "hipEventRecord failed");
        }
        ++n;
        return MA_OK;
    }
};

// Untyped tensors and states of one call (the states are null on the fused
// path; obj_part and obj are null unless the objective is requested).
struct CallBufs {
    const void *q, *k, *v;
    void *out;
    void *aR, *aL, *Y;
    float *cR, *cL;
    float *obj_part;  // [B*H][T][b] shares (workspace)
    float *obj;       // [B*H][T] result (caller's)
    const int *lens = nullptr;  // [B] real rows per batch element (device), or null
    int rev = 0;                // pre-padded sequences (HeadDims::rev)
};

struct CallDims {
    int64_t BH;
    int64_t H;  // heads per batch element
    int m, b, n, d, T;  // n: rows per head, (m - 1) * b < n <= m * b
    float s_log2e;
    int num_cus;  // compute units of the device
};

// Path selection (monarch_attn_set_path): 0 = automatic; 1 = one launch per
// half-step; 2 = one workgroup per head (or MA_EUNSUPPORTED); 3 = one
// workgroup per (head, group of residue classes) (or MA_EUNSUPPORTED).
enum Path { kAuto = 0, kHalfSteps = 1, kFusedHead = 2, kGrouped = 3 };

// The kernel family that runs a forward call.
enum Family { kFamHalf = 0, kFamFused = 1, kFamGroup = 2, kFamNone = -1 };

// Tile width of the kernels for head dimension d (columns d..D-1 are zero).
inline int tile_d(int64_t d) { return d <= 64 ? 64 : d <= 96 ? 96 : 128; }

// The fused one-workgroup-per-head kernel holds Q, K and all states of a head
// in LDS: 16-bit elements, d <= 64, m and b at most 16.
inline bool fused_applies(int32_t dtype, int64_t d, int64_t m, int64_t b)
{
    return (dtype == MA_BF16 || dtype == MA_F16) && d <= 64 && m <= 16 && b <= 16;
}

// The one-workgroup-per-(head, group of classes) kernel keeps the states of
// its classes in LDS: 16-bit elements, d <= 64, m at most 64, b at most 32,
// and neither per-sequence lengths nor the objective.
inline bool grouped_applies(int32_t dtype, int64_t d, int64_t m, int64_t b, bool lens, bool obj)
{
    return (dtype == MA_BF16 || dtype == MA_F16) && d <= 64 && m <= 64 && b <= 32 && !lens && !obj;
}

// Heads of up to 16 blocks of up to 16 rows.
inline bool small_heads(int32_t dtype, int64_t m, int64_t b)
{
    return (dtype == MA_BF16 || dtype == MA_F16) && m <= 16 && b <= 16;
}

// Whether heads that take a compute unit each, in rounds of num_cus, are large
// enough for their rounds: one of few units (m + b, which the half-steps run a
// dozen a compute unit) leaves it idle.  Any up to `free` rounds; from 16 units
// up always; between them `base` units and `quarters` / 4 a round, begun rounds
// counting whole.
inline bool fills_rounds(int64_t BH, int64_t units, int64_t num_cus, int64_t free, int64_t base, int64_t quarters)
{
    const int64_t rounds = (BH + num_cus - 1) / num_cus;
    return rounds <= free || units >= 16 || 4 * (units - base) >= quarters * rounds;
}

// Small heads that the automatic path gives to the half-steps (d > 64, beyond
// fused_applies): whether the half-steps' launches are one of the
// one-workgroup-per-head kernel, which takes any d (the workspace rules stay
// those of the half-steps).  Times against the half-steps':
// - one step of few large heads, which two launches spread over m and b
//   workgroups a head: at 128 columns, 4 heads: 16 x 16 rows 1.19 (8.5 us),
//   15 x 14 1.11, 16 x 4 0.99, 8 x 8 0.94, with lengths 1.22, 1.16, 1.03, 1.00;
//   24 heads of 16 x 16 1.01, 32 heads 0.95.  At 96 columns 16 x 16 rows 1.06
//   for 4 heads, 1.01 for 12, 0.94 for 24; smaller heads 0.85 to 0.99;
// - one step of many tiny heads (d = 72; at 128 columns up to 0.1 more): 512
//   heads of 2, 6 and 9 units 1.11, 0.98 and 0.90, but 290 to 320 heads of 9
//   units 1.06 to 1.11; 1024 heads of 8, 10 and 12 units 1.10, 1.02 and 0.87;
//   4096 heads of 12, 16 and 17 units 1.21, 0.88 and 0.95 to 1.08;
// - two steps: 0.3 to 0.7 up to 512 heads; 1024 heads of 3, 6 and 8 units 1.16,
//   0.91 and 0.76; 4096 heads of 8, 10, 12 and 17 units 1.17, 1.05, 0.90, 0.76.
//   Three steps: 1024 heads of 3 and 5 units 0.97 and 0.83; 4096 heads of 6, 8
//   and 9 units 1.17, 1.00 and 0.95.
inline bool one_launch_forward(int64_t BH, int64_t d, int64_t m, int64_t b, int T, bool lens, int64_t num_cus)
{
    const bool wide = tile_d(d) == 128;
    const int64_t rows = wide ? (lens ? 64 : 144) : 256;
    if (T == 1 && m * b >= rows && BH < (wide ? 24 : 12)) return false;
    return T == 1 ? fills_rounds(BH, m + b, num_cus, 1, 8, 4) : fills_rounds(BH, m + b, num_cus, 2, T == 2 ? 6 : 4, 1);
}

// The same for the gradient's recompute, at any d.  One step is one launch on
// the half-steps too, of m workgroups a head: the whole gradient takes 1.0 to
// 1.4 times as long with one (4 to 256 heads; 1.0 to 1.17 from 384 to 2048).
// Two steps are three launches: 0.85 to 1.0 of the gradient up to 256 heads, but
// - few large heads (1 to 63): at 128 columns 16 x 16 rows 1.02 to 1.10, 15 x 14
//   1.02 to 1.09, 16 x 8 0.99 to 1.04, 16 x 4 0.96 to 1.01, 8 x 8 0.97; at 96
//   columns 16 x 16 rows 1.03 to 1.05, 15 x 14 0.98 (100 heads: 0.98 at most);
// - many tiny heads: 512 heads of 2, 8 and 10 units 0.97 to 1.09, 0.98 to 1.02
//   and 0.97 to 1.02; 1024 heads of 6, 10 and 12 units 1.07 to 1.14, 1.05 and
//   1.00 to 1.02; 4096 heads of 2, 12, 16 and 18 units 1.7, 1.05, 1.00 and 1.02.
// Three steps: up to 512 heads 0.82 to 1.03; 1024 heads of 6 and 8 units 1.01 to
// 1.06 and 0.98 to 1.02; 4096 heads of 10, 12 and 16 units 1.05, 1.02 and 0.97.
inline bool one_launch_recompute(int64_t BH, int64_t d, int64_t m, int64_t b, int T, int64_t num_cus)
{
    const int D = tile_d(d);
    if (T == 1 || (T == 2 && BH < 64 && D > 64 && m * b >= (D == 128 ? 128 : 256))) return false;
    return T == 2 ? fills_rounds(BH, m + b, num_cus, 1, 6, 8) : fills_rounds(BH, m + b, num_cus, 2, 4, 4);
}

// The family that runs a call under `path` (kFamNone: the forced path does
// not take the shape).  Automatic: the one-workgroup-per-head kernel where it
// applies; else the grouped kernel where it applies with m <= 32 (measured
// faster than the half-steps there at 16 and 192 heads and T = 1, 2, apart
// from 24-row blocks at T = 1 with many heads, up to 15% slower; with more
// blocks every group streams more of K and V); else the half-steps.  All
// families give the same bits.
inline int family_of(int path, int32_t dtype, int64_t d, int64_t m, int64_t b, bool lens, bool obj)
{
    switch (path) {
    case kHalfSteps: return kFamHalf;
    case kFusedHead: return fused_applies(dtype, d, m, b) ? kFamFused : kFamNone;
    case kGrouped: return grouped_applies(dtype, d, m, b, lens, obj) ? kFamGroup : kFamNone;
    default:
        if (fused_applies(dtype, d, m, b)) return kFamFused;
        if (grouped_applies(dtype, d, m, b, lens, obj) && m <= 32) return kFamGroup;
        return kFamHalf;
    }
}

// Enqueue the whole forward pass for one element type (defined per dtype).
template <typename T> int run_call(Launcher &L, const CallBufs &B, const CallDims &c, int path);

// Buffers of one gradient call: the caller's tensors, the states of every
// step of the recomputed forward pass (alpha_R and c_R of steps 2..T, alpha_L
// and c_L of steps 1..T, `st` bytes resp. `cst` floats apart, and Y), and the
// fp32 gradients of the states and accumulators of dQ, dK.
struct BwdCallBufs {
    const void *q, *k, *v, *dout;
    void *dq, *dk, *dv;
    char *aR, *aL;
    void *Y;
    float *cR, *cL;
    size_t st, cst;
    float *dQ, *dK, *daL, *dcL, *dY, *daR, *dcR;
    const int *lens = nullptr;  // [B] real rows per batch element (device), or null
    int path = kAuto;
};

// The gradient's reverse sweep for one element type and tile width (sweep_*.hip).
template <typename T, int D> int bwd_sweep(Launcher &L, const BwdCallBufs &B, const CallDims &c);

// Enqueue the gradient (forward recompute, then the reverse sweep) for one
// element type; under a forced path the recompute runs the half-steps.
template <typename T> int run_bwd(Launcher &L, const BwdCallBufs &B, const CallDims &c);

// Enqueue exact softmax attention (with the row logsumexps when lse != null).
template <typename T> int run_exact(Launcher &L, const CallBufs &B, float *lse, int64_t BH, int n, int d);

}  // namespace ma_host
