// Launches of the brick kernels, one translation unit per storage type
// (lbm_brick_<storage>.hip).
#pragma once

#include "lbm_brick.hpp"
#include "lbm_launch.hpp"

namespace lbm_host {

using namespace lbm;

template <int S, int RX, int RY, int MODE>
hipError_t launch_brick_t(const KParams<typename Traits<S>::C> &p, int steps, int tiles_x, hipStream_t st)
{
    const int per_xcd = (p.n_units + 7) / 8;
    hipLaunchKernelGGL((k_brick<S, RX, RY, MODE>), dim3(per_xcd * 8), dim3((RX * RY + 63) / 64 * 64), 0, st, p, steps,
                       tiles_x, per_xcd);
    return hipGetLastError();
}

template <int S, int MODE>
hipError_t launch_brick_m(KParams<typename Traits<S>::C> &p, int region, int steps, hipStream_t st)
{
    const int w = brick_core(brick_rx(region), steps), h = brick_core(brick_ry(region), steps);
    if (w < 1 || h < 1) return hipErrorInvalidValue;
    const int tiles_x = (p.nx + w - 1) / w, tiles_y = (p.ny + h - 1) / h;
    p.n_units = tiles_x * tiles_y;
    if (region == 0) return launch_brick_t<S, brick_rx(0), brick_ry(0), MODE>(p, steps, tiles_x, st);
    // (FP64 with boundary code has no registers for the larger region)
    if constexpr (S == ST_F64 && (MODE & M_BND)) return hipErrorInvalidValue;
    else return launch_brick_t<S, brick_rx(1), brick_ry(1), MODE>(p, steps, tiles_x, st);
}

template <int S>
hipError_t launch_brick(KParams<typename Traits<S>::C> p, int region, int steps, bool sr, bool bnd, hipStream_t st)
{
    if constexpr (S == ST_F16 || S == ST_BF16) {
        if (sr)
            return bnd ? launch_brick_m<S, M_SR | M_BND>(p, region, steps, st) : launch_brick_m<S, M_SR>(p, region, steps, st);
    }
    return bnd ? launch_brick_m<S, M_BND>(p, region, steps, st) : launch_brick_m<S, 0>(p, region, steps, st);
}

}  // namespace lbm_host
