#include "gemm_mfma.h"

namespace t5mi {

hipError_t launch_gemm_mfma_geglu_fwd(const GemmDesc& g, const GemmEpi& e, hipStream_t st) {
  return e.drop.on ? launch_layout<true, true, EPI_GEGLU_FWD | EPI_DROP>(g, e, st) : launch_layout<true, true, EPI_GEGLU_FWD>(g, e, st);
}

}  // namespace t5mi
