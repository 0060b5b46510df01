// Step-kernel instances of relaxation time 1 for F16 storage (see lbm_launch.hpp).
#include "lbm_launch_impl.hpp"

namespace lbm_host {
template hipError_t launch_tau1<lbm::ST_F16>(const lbm::KParams<float> &, Pass, int, bool, bool, hipStream_t);
}  // namespace lbm_host
