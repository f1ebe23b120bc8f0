// The register-weight GEMM, fp32 split-K partials.
#include "gemm_wide.hpp"

namespace hxf {

hipError_t gemm_wide_split(const GemmArgs& a, const GemmPlan& p, hipStream_t st, hipEvent_t e0, hipEvent_t e1) {
  if (!a.B2) return launch_wide_cfg<EPI_F32, true>(a, p, st, e0, e1);
  switch (p.nw == 2 ? p.tm : 0) {   // SwiGLU
    case 1: return launch_wide<1, 2, 4, 2, EPI_SWIGLU, true>(a, p, st, e0, e1);
    case 2: return launch_wide<2, 2, 4, 2, EPI_SWIGLU, true>(a, p, st, e0, e1);
    case 4: return launch_wide<4, 2, 4, 2, EPI_SWIGLU, true>(a, p, st, e0, e1);
    case 8: return launch_wide<8, 2, 4, 2, EPI_SWIGLU, true>(a, p, st, e0, e1);
  }
  return hipErrorInvalidValue;
}

}  // namespace hxf
