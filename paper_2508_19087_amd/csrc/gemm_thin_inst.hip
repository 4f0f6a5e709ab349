// gemm_thin_inst.hip - instantiates the few-token GEMM kernels for one weight
// bit width, APT_INST_P (the build compiles this file once per width).
#include "gemm_thin.h"

namespace apt {
namespace thin {

template <int P>
hipError_t launch_for_p(const ThinParams& prm, const ThinLaunch& L, hipStream_t s) {
  const bool fused = prm.src != kSrcPacked;
  if constexpr (P <= 4) {
    if (L.cls == kLow) return fused ? launch_cls<P, kLow, true>(prm, L, s) : launch_cls<P, kLow, false>(prm, L, s);
  }
  if (fused) return launch_cls<P, kByte, true>(prm, L, s);
  if (L.cls == kByte) return launch_cls<P, kByte, false>(prm, L, s);
  if (L.cls == kByte8) return launch_cls<P, kByte8, false>(prm, L, s);
  return hipErrorInvalidValue;
}

template hipError_t launch_for_p<APT_INST_P>(const ThinParams&, const ThinLaunch&, hipStream_t);

}  // namespace thin
}  // namespace apt
