// The one-workgroup-per-head kernel for element type _Float16.
#include "dispatch_fused.hpp"

namespace ma_host {
template int run_fused<_Float16>(Launcher &L, const CallBufs &B, ma::HeadDims hd, const CallDims &c);
template int run_fused_states<_Float16>(Launcher &L, const CallBufs &B, ma::HeadDims hd, const CallDims &c, int64_t st,
                                  int64_t cst);
}  // namespace ma_host
