#include "gemm_mfma.h"

namespace t5mi {

hipError_t launch_gemm_mfma_store(const GemmDesc& g, const GemmEpi& e, hipStream_t st) {
  return e.drop.on ? launch_layout<true, true, EPI_STORE | EPI_DROP>(g, e, st) : launch_layout<true, true, EPI_STORE>(g, e, st);
}

}  // namespace t5mi
