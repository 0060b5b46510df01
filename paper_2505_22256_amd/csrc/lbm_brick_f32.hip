// Brick kernel instances for F32 storage (see lbm_launch.hpp).
#include "lbm_brick_impl.hpp"

namespace lbm_host {
template hipError_t launch_brick<lbm::ST_F32>(lbm::KParams<float>, int, int, bool, bool, hipStream_t);
}  // namespace lbm_host
