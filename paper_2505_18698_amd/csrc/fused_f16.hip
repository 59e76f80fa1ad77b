// The one-workgroup-per-head kernel for element type _Float16.
#include "dispatch_fused.hpp"

namespace ma_host {
template int run_fused<_Float16>(Launcher &L, const CallBufs &B, ma::HeadDims hd, const CallDims &c);
}  // namespace ma_host
