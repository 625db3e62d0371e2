#include "gemm_mfma.h"

namespace t5mi {

hipError_t launch_gemm_mfma_resid(const GemmDesc& g, const GemmEpi& e, hipStream_t st) {
  return e.drop.on ? launch_layout<true, true, EPI_RESID | EPI_DROP>(g, e, st) : launch_layout<true, true, EPI_RESID>(g, e, st);
}

}  // namespace t5mi
