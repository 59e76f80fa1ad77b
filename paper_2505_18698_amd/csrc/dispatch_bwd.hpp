// Launches of the gradient's reverse sweep (backward.hpp).  Instantiated once
// per element type and tile width in sweep_{bf16,f16,f32}_{64,96,128}.hip, so
// that the kernels compile in parallel.
#pragma once

#include <cmath>
#include <type_traits>

#include "backward.hpp"
#include "host_common.hpp"

namespace ma_host {

// ---- gradient ----
template <typename T, int S, int D, bool LAST, bool LENS>
int launch_l_bwd(Launcher &L, const ma::BwdBufs<T> &p, const ma::BwdDims &dm, int64_t BH)
{
    const dim3 grid((unsigned)(BH * dm.b)), block(ma::bwd::unit_threads<T, S, D, true, LAST>);
    return L.run(kBwdL, [&] {
        return launched(
            [&] { hipLaunchKernelGGL((ma::bwd::l_bwd<T, S, D, LAST, LENS>), grid, block, 0, L.stream, p, dm); });
    });
}

template <typename T, int S, int D, bool FIRST, bool LAST, bool LENS>
int launch_r_bwd(Launcher &L, const ma::BwdBufs<T> &p, const ma::BwdDims &dm, int64_t BH)
{
    const dim3 grid((unsigned)(BH * dm.m)), block(ma::bwd::unit_threads<T, S, D, false, LAST>);
    return L.run(kBwdR, [&] {
        return launched(
            [&] { hipLaunchKernelGGL((ma::bwd::r_bwd<T, S, D, FIRST, LAST, LENS>), grid, block, 0, L.stream, p, dm); });
    });
}

// One launch of the L-update gradient of a step, on tiles of S >= m rows (and
// of the R-update gradient, S >= b): each kernel takes the tile of its own
// dimension.
template <typename T, int D, bool LENS>
int l_bwd_step(Launcher &L, const ma::BwdBufs<T> &p, const ma::BwdDims &dm, int64_t BH, bool last)
{
    switch (tile_rows(dm.m)) {
    case 16: return last ? launch_l_bwd<T, 16, D, true, LENS>(L, p, dm, BH) : launch_l_bwd<T, 16, D, false, LENS>(L, p, dm, BH);
    case 32: return last ? launch_l_bwd<T, 32, D, true, LENS>(L, p, dm, BH) : launch_l_bwd<T, 32, D, false, LENS>(L, p, dm, BH);
    case 64: return last ? launch_l_bwd<T, 64, D, true, LENS>(L, p, dm, BH) : launch_l_bwd<T, 64, D, false, LENS>(L, p, dm, BH);
    default:
        if constexpr (D > 64 && std::is_same<T, float>::value) {  // the forward takes no such fp32 shape
            return fail(MA_EUNSUPPORTED, "fp32 128-row blocks need d <= 64");
        } else {
            return last ? launch_l_bwd<T, 128, D, true, LENS>(L, p, dm, BH)
                        : launch_l_bwd<T, 128, D, false, LENS>(L, p, dm, BH);
        }
    }
}

template <typename T, int S, int D, bool LENS>
int r_bwd_tile(Launcher &L, const ma::BwdBufs<T> &p, const ma::BwdDims &dm, int64_t BH, bool first, bool last)
{
    if (first)
        return last ? launch_r_bwd<T, S, D, true, true, LENS>(L, p, dm, BH)
                    : launch_r_bwd<T, S, D, true, false, LENS>(L, p, dm, BH);
    return last ? launch_r_bwd<T, S, D, false, true, LENS>(L, p, dm, BH)
                : launch_r_bwd<T, S, D, false, false, LENS>(L, p, dm, BH);
}

template <typename T, int D, bool LENS>
int r_bwd_step(Launcher &L, const ma::BwdBufs<T> &p, const ma::BwdDims &dm, int64_t BH, bool first, bool last)
{
    switch (tile_rows(dm.b)) {
    case 16: return r_bwd_tile<T, 16, D, LENS>(L, p, dm, BH, first, last);
    case 32: return r_bwd_tile<T, 32, D, LENS>(L, p, dm, BH, first, last);
    case 64: return r_bwd_tile<T, 64, D, LENS>(L, p, dm, BH, first, last);
    default:
        if constexpr (D > 64 && std::is_same<T, float>::value) {  // the forward takes no such fp32 shape
            return fail(MA_EUNSUPPORTED, "fp32 128-row blocks need d <= 64");
        } else {
            return r_bwd_tile<T, 128, D, LENS>(L, p, dm, BH, first, last);
        }
    }
}

// The reverse sweep, t = T .. 1: the L update of step t, then its R update.
// LENS: per-sequence lengths (instantiations of their own).
template <typename T, int D, bool LENS> int bwd_sweep_impl(Launcher &L, const BwdCallBufs &B, const CallDims &c)
{
    ma::BwdDims dm{c.m, c.b, c.n, c.d, (float)(1.0 / std::sqrt((double)c.d))};
    dm.lens = B.lens;
    dm.H = (int)c.H;
    ma::BwdBufs<T> p{(const T *)B.q, (const T *)B.k, (const T *)B.v, (const T *)B.dout, nullptr, nullptr,
                     (const T *)B.Y, nullptr, nullptr, B.dQ, B.dK, (T *)B.dq, (T *)B.dk, (T *)B.dv, B.daL, B.dcL,
                     B.dY, B.daR, B.dcR};
    int rc;
    for (int t = c.T; t >= 1; --t) {
        const bool first = t == 1, last = t == c.T;
        p.aL = (const T *)(B.aL + (size_t)(t - 1) * B.st);
        p.cL = B.cL + (size_t)(t - 1) * B.cst;
        p.aR = first ? nullptr : (const T *)(B.aR + (size_t)(t - 2) * B.st);
        p.cR = first ? nullptr : B.cR + (size_t)(t - 2) * B.cst;
        if ((rc = l_bwd_step<T, D, LENS>(L, p, dm, c.BH, last)) != MA_OK) return rc;
        if ((rc = r_bwd_step<T, D, LENS>(L, p, dm, c.BH, first, last)) != MA_OK) return rc;
    }
    return MA_OK;
}

template <typename T, int D> int bwd_sweep(Launcher &L, const BwdCallBufs &B, const CallDims &c)
{
    return B.lens ? bwd_sweep_impl<T, D, true>(L, B, c) : bwd_sweep_impl<T, D, false>(L, B, c);
}

}  // namespace ma_host
