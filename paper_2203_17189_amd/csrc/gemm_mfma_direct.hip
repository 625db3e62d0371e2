// The forward products of a few hundred tokens with the weights as the caller stores them ([K, N], columns of up to three
// matrices side by side): A k-contiguous, B read through the LDS transpose.  Packing the weights first (transposed copies,
// 4 bytes moved per weight) pays where many row tiles read a weight; below, it is a tenth of the forward and more (d 768,
// 1332 tokens: 76 -> 69 us, d 2048, 128 tokens: 117 -> 89).
#include "gemm_mfma.h"

namespace t5mi {

bool gemm_direct_supported(const GemmDesc& g, const GemmEpi& e) {
  if (g.in_type != IN_BF16 || !g.a_kc || g.b_kc || g.nseg != 1 || g.ngroups > 1 || e.drop.on) return false;
  const GemmSeg& sg = g.seg[0];
  const int nsrc = g.nsrc > 1 ? g.nsrc : 1, cols = nsrc > 1 ? g.nsrc_cols : g.N;
  if (sg.K < KQ || sg.K % KQ != 0 || cols % 64 != 0 || nsrc > 3 || nsrc * cols != g.N || g.M < 8) return false;
  if (sg.lda % 8 != 0 || sg.ldb % 8 != 0 || ((uintptr_t)sg.A & 15)) return false;
  // the lanes' 32-bit byte offsets reach from the lowest matrix to the last rows of a k-tile in the highest
  uint64_t lo = ~0ull, hi = 0;
  for (int s = 0; s < nsrc; ++s) {
    const uint64_t p = (uint64_t)g.seg[s].B;
    if (p & 15) return false;
    lo = p < lo ? p : lo;
    hi = p > hi ? p : hi;
  }
  if (hi - lo + (uint64_t)(KQ + 1) * sg.ldb * 2 >= (1ull << 32) || (uint64_t)g.M * sg.lda * 2 >= (1ull << 32)) return false;
  switch (e.kind) {
    case EPI_STORE: case EPI_RESID: return true;
    case EPI_GEGLU_FWD: return nsrc == 2 && e.out_type == IN_BF16;
    default: return false;
  }
}

namespace {

template <int EPI>
hipError_t launch_direct(const GemmDesc& g, const GemmEpi& e, hipStream_t st) {
  // the tiles that packed weights get at these sizes (launch_layout)
  if ((int64_t)ceil_div(g.M, 128) * ceil_div(g.N, 128) <= 256) {
    if constexpr (EPI != EPI_GEGLU_FWD) {
      if ((int64_t)ceil_div(g.M, 64) * ceil_div(g.N, 64) <= 256) return launch_cfg<64, 64, 1, 2, true, false, EPI, 4, 1, 64>(g, e, 1, st);
      if ((int64_t)ceil_div(g.M, 128) * ceil_div(g.N, 64) <= 256) return launch_cfg<128, 64, 2, 2, true, false, EPI, 3, 1, 64>(g, e, 1, st);
    }
    // Four stages of 64 from K = 1536 on, with residual from above 1024 (us in a layer's forward with stages of 32 and with these.
    // Residual, N = 768, 4000 rows: K 1280 21.1 and 20.4, 1536 23.2 and 22.2, 1792 25.4 and 23.9, 2048 28.1 and 25.9; N = 1024, 3500
    // rows: 21.1 and 20.1, 23.4 and 21.9, 25.6 and 23.5, 28.1 and 25.0; 1024 in two runs 18.1 and 16.9, 18.6 and 20.5.  Queries,
    // keys and values, N = 768, 5200 rows: 1024 14.4 and 14.8, 1280 16.8 and 16.4, 1536 18.8 and 17.9, 2048 22.1 and 21.2; 4000 rows: 1024
    // 13.8 and 14.4, 1280 15.6 and 16.0, 1536 17.6 and 17.3, 2048 20.4 and 20.0.  Gated, N = 768, 4000 rows: 1024 14.8 and 15.3, 1280
    // 16.2 and 16.8, 1536 17.9 and 17.7, 2048 21.1 and 20.1).
    if (g.seg[0].K >= 1536 || (EPI == EPI_RESID && g.seg[0].K > 1024))
      return launch_cfg<128, 128, 2, 2, true, false, EPI, 4, 1, 64>(g, e, 1, st);
    return launch_cfg<128, 128, 2, 2, true, false, EPI, 4, 1>(g, e, 1, st);
  }
  // (three stages of A and two of B lose here: 8192 x 2048 x 512 gated 32 -> 37 us)
  return launch_cfg<128, 128, 2, 2, true, false, EPI, 2, 1, 64>(g, e, 1, st);
}

}  // namespace

hipError_t launch_gemm_direct(const GemmDesc& g, const GemmEpi& e, hipStream_t st) {
  switch (e.kind) {
    case EPI_STORE: return launch_direct<EPI_STORE>(g, e, st);
    case EPI_RESID: return launch_direct<EPI_RESID>(g, e, st);
    case EPI_GEGLU_FWD: return launch_direct<EPI_GEGLU_FWD>(g, e, st);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace t5mi
