// Launch helpers shared by the dispatch units.
#pragma once

#include <mutex>
#include <unordered_map>

#include "host_common.hpp"
#include "ma_kernels.hpp"

namespace ma_host {

template <typename T> ma::Bufs<T> typed(const CallBufs &B)
{
    return ma::Bufs<T>{(const T *)B.q, (const T *)B.k, (const T *)B.v, (T *)B.out, (T *)B.aR, (T *)B.aL, (T *)B.Y,
                       B.cR, B.cL, B.obj_part};
}

// Workgroups of `kern` (at `threads` threads) resident on one compute unit,
// queried once per kernel.
inline int resident_per_cu(const void *kern, int threads)
{
    static std::mutex mu;
    static std::unordered_map<const void *, int> cache;
    std::lock_guard<std::mutex> lock(mu);
    auto it = cache.find(kern);
    if (it != cache.end()) return it->second;
    int n = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, kern, threads, 0) != hipSuccess || n < 1) {
        (void)hipGetLastError();
        n = 1;
    }
    cache.emplace(kern, n);
    return n;
}

// The forward pass of heads with m, b <= 16, one workgroup per head (fused_*.hip; 16-bit elements).
template <typename T> int run_fused(Launcher &L, const CallBufs &B, ma::HeadDims hd, const CallDims &c);

// The same heads' states of every step (the gradient's recompute), `st`
// elements resp. `cst` floats from step to step.
template <typename T>
int run_fused_states(Launcher &L, const CallBufs &B, ma::HeadDims hd, const CallDims &c, int64_t st, int64_t cst);

}  // namespace ma_host
