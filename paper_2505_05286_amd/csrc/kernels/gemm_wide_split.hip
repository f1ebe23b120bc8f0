// The register-weight GEMM, fp32 split-K partials.
#include "gemm_wide.hpp"

namespace hxf {

hipError_t gemm_wide_split(const GemmArgs& a, const GemmPlan& p, hipStream_t st, hipEvent_t e0, hipEvent_t e1) {
  return launch_wide_cfg<EPI_F32, true>(a, p, st, e0, e1);
}

}  // namespace hxf
