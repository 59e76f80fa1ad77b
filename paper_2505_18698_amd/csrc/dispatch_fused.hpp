// Launches of the one-workgroup-per-head kernel (fused.hpp).  Instantiated once
// per 16-bit element type in fused_{bf16,f16}.hip.
#pragma once

#include "fused.hpp"
#include "launch.hpp"

namespace ma_host {

// One workgroup a head, or as many as are resident at once, each looping over heads.
template <typename U> dim3 head_grid(const void *kern, const CallDims &c)
{
    if (!U::LOOP) return c.BH <= U::ROW ? dim3((unsigned)c.BH) : dim3(U::ROW, (unsigned)((c.BH + U::ROW - 1) / U::ROW));
    const int64_t cap = (int64_t)resident_per_cu(kern, U::NTH) * c.num_cus;
    return dim3((unsigned)(c.BH < cap ? c.BH : cap));
}

template <typename T, int D, bool RGB, bool RGM, bool LENS = false>
int launch_fused(Launcher &L, const CallBufs &B, const ma::HeadDims &hd, const CallDims &c)
{
    using U = ma::FusedHead<T, D, RGB, RGM, LENS>;
    auto kern = ma::monarch_fused_head<T, D, RGB, RGM, LENS>;
    const dim3 grid = head_grid<U>((const void *)kern, c);
    const ma::Bufs<T> p = typed<T>(B);
    const int64_t BH = c.BH;
    const int T_ = c.T;
    return L.run(kFused, [&] {
        return launched([&] { hipLaunchKernelGGL(kern, grid, dim3(U::NTH), 0, L.stream, p, hd, BH, T_); });
    });
}

template <typename T, int D, bool RGB, bool RGM, bool LENS = false>
int launch_states(Launcher &L, const CallBufs &B, const ma::HeadDims &hd, const CallDims &c, const ma::KeptStates<T> &keep)
{
    using U = ma::FusedHead<T, D, RGB, RGM, LENS, true>;
    auto kern = ma::monarch_fused_states<T, D, RGB, RGM, LENS>;
    const dim3 grid = head_grid<U>((const void *)kern, c);
    const ma::Bufs<T> p = typed<T>(B);
    const int64_t BH = c.BH;
    const int T_ = c.T;
    return L.run(kFused, [&] {
        return launched([&] { hipLaunchKernelGGL(kern, grid, dim3(U::NTH), 0, L.stream, p, hd, BH, T_, keep); });
    });
}

template <typename T, int D>
int run_states_d(Launcher &L, const CallBufs &B, ma::HeadDims hd, const CallDims &c, const ma::KeptStates<T> &keep)
{
    if (hd.lens) return launch_states<T, D, true, true, true>(L, B, hd, c, keep);
    const bool rgb = hd.b != 16 || hd.n != hd.m * hd.b, rgm = hd.m != 16;
    if (rgb && rgm) return launch_states<T, D, true, true>(L, B, hd, c, keep);
    if (rgb) return launch_states<T, D, true, false>(L, B, hd, c, keep);
    if (rgm) return launch_states<T, D, false, true>(L, B, hd, c, keep);
    return launch_states<T, D, false, false>(L, B, hd, c, keep);
}

template <typename T>
int run_fused_states(Launcher &L, const CallBufs &B, ma::HeadDims hd, const CallDims &c, int64_t st, int64_t cst)
{
    const ma::KeptStates<T> keep{(T *)B.aR, (T *)B.aL, (T *)B.Y, B.cR, B.cL, st, cst};
    switch (tile_d(c.d)) {
    case 64: return run_states_d<T, 64>(L, B, hd, c, keep);
    case 96: return run_states_d<T, 96>(L, B, hd, c, keep);
    default: return run_states_d<T, 128>(L, B, hd, c, keep);
    }
}

template <typename T, int D> int run_fused_d(Launcher &L, const CallBufs &B, ma::HeadDims hd, const CallDims &c)
{
    if (hd.lens) return launch_fused<T, D, true, true, true>(L, B, hd, c);
    const bool rgb = hd.b != 16 || hd.n != hd.m * hd.b, rgm = hd.m != 16;
    if (rgb && rgm) return launch_fused<T, D, true, true>(L, B, hd, c);
    if (rgb) return launch_fused<T, D, true, false>(L, B, hd, c);
    if (rgm) return launch_fused<T, D, false, true>(L, B, hd, c);
    return launch_fused<T, D, false, false>(L, B, hd, c);
}

template <typename T> int run_fused(Launcher &L, const CallBufs &B, ma::HeadDims hd, const CallDims &c)
{
    switch (tile_d(c.d)) {
    case 64: return run_fused_d<T, 64>(L, B, hd, c);
    case 96: return run_fused_d<T, 96>(L, B, hd, c);
    default: return run_fused_d<T, 128>(L, B, hd, c);
    }
}

}  // namespace ma_host
