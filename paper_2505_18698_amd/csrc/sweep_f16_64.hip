// The gradient's reverse sweep for element type _Float16 at tile width 64.
#include "dispatch_bwd.hpp"

namespace ma_host {
template int bwd_sweep<_Float16, 64>(Launcher &L, const BwdCallBufs &B, const CallDims &c);
}  // namespace ma_host
