#include "gemm_mfma.h"

namespace t5mi {

hipError_t launch_gemm_mfma_geglu_bwd(const GemmDesc& g, const GemmEpi& e, hipStream_t st) {
  return launch_layout<true, true, EPI_GEGLU_BWD>(g, e, st);
}

}  // namespace t5mi
