// gemm_direct_inst.hip - instantiates the direct-weight MFMA kernel for one
// weight bit width, APT_INST_P (the build compiles this file once per width;
// widths above 4 have none).
#include "gemm_direct.h"

namespace apt {
namespace direct {

#if APT_INST_P <= 4
template <int P>
hipError_t launch_for_p(const Int8Params& prm, hipStream_t s) {
  return launch_kernel(gemm_direct_kernel<P>, dim3(prm.tiles), dim3(kWaves * kWave), 0, s, prm);
}

template hipError_t launch_for_p<APT_INST_P>(const Int8Params&, hipStream_t);
#endif

}  // namespace direct
}  // namespace apt
