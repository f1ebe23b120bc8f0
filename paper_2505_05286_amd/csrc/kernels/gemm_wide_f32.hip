// The register-weight GEMM, fp32 output.
#include "gemm_wide.hpp"

namespace hxf {

hipError_t gemm_wide_f32(const GemmArgs& a, const GemmPlan& p, hipStream_t st, hipEvent_t e0, hipEvent_t e1) {
  return launch_wide_cfg<EPI_F32, false>(a, p, st, e0, e1);
}

}  // namespace hxf
