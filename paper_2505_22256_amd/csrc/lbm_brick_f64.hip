// Brick kernel instances for F64 storage (see lbm_launch.hpp).
#include "lbm_brick_impl.hpp"

namespace lbm_host {
template hipError_t launch_brick<lbm::ST_F64>(lbm::KParams<double>, int, int, bool, bool, hipStream_t);
}  // namespace lbm_host
