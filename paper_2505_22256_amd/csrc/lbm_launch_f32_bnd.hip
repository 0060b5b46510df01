// Step-kernel instances with boundary code for F32 storage (see lbm_launch.hpp).
#include "lbm_launch_impl.hpp"

namespace lbm_host {
template hipError_t launch_pass_b<lbm::ST_F32, lbm::M_BND>(const lbm::KParams<float> &, Pass, int, bool, hipStream_t, bool);
}  // namespace lbm_host
