#include "gemm_mfma.h"

namespace t5mi {

hipError_t launch_gemm_mfma_split(const GemmDesc& g, const GemmEpi& e, hipStream_t st) {
  return launch_layout<false, false, EPI_SPLIT_F32>(g, e, st);
}

}  // namespace t5mi
