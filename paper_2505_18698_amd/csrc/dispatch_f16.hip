// Kernels and dispatch for element type _Float16.
#include "dispatch.hpp"

namespace ma_host {
template <> int run_call<_Float16>(Launcher &L, const CallBufs &B, const CallDims &c, int path)
{
    return run_call_impl<_Float16>(L, B, c, path);
}
template <> int run_exact<_Float16>(Launcher &L, const CallBufs &B, float *lse, int64_t BH, int n, int d)
{
    return run_exact_impl<_Float16>(L, B, lse, BH, n, d);
}
template <> int run_bwd<_Float16>(Launcher &L, const BwdCallBufs &B, const CallDims &c)
{
    return run_bwd_impl<_Float16>(L, B, c);
}
}  // namespace ma_host
