// Walks the choice between the two places that the attention kernels take their bias from (tests/test_attention_plan.py).
#include <cstdio>
#include <cstring>
#include "../../paper_2203_17189_amd/csrc/kernels.h"

using namespace t5mi;

int main() {
  int failures = 0, windows = 0, slices = 0;
  const int fars[] = {1, 31, 33, 64, 65, 91, 97, 113, 128, 130, 165, 166, 200, 216, 225, 226, 300, 413, 449, 450, 700};
  for (int dk = 64; dk <= 128; dk += 64)
    for (int causal = 0; causal < 2; ++causal)
      for (int drop = 0; drop < 2; ++drop)
        for (int far : fars)
          for (int S = 32; S <= 8192; S += S < 600 ? 7 : 331) {
            AttnDims a;
            std::memset(&a, 0, sizeof(a));
            a.B = 1; a.H = 1; a.S = a.Sk = S; a.dk = dk; a.causal = causal; a.bias = 1; a.drop.on = drop; a.far = far;
            if (!attn_mfma_supported(a) || !attn_bwd_mfma_fits(a)) continue;
            for (AttnPass pass : {ATTN_FWD, ATTN_BWD_DQ, ATTN_BWD_DKV}) {
              const bool window = attn_bias_window(a, pass);
              ++(window ? windows : slices);
              const int here = attn_workgroups_per_unit(a, pass, window), slice = attn_workgroups_per_unit(a, pass, false);
              const int least = pass == ATTN_BWD_DKV && dk == 64 ? 2 : 1;
              if (here < least || here < slice || attn_lds_bytes(a, pass, window) > 160 * 1024) {
                if (++failures <= 20)
                  std::printf("dk %d causal %d dropout %d far %d S %d pass %d: window %d, %d workgroups a unit (slice %d)\n", dk,
                              causal, drop, far, S, (int)pass, (int)window, here, slice);
              }
            }
          }
  std::printf("%d failure(s), %d windows, %d slices\n", failures, windows, slices);
  return failures || !windows || !slices;
}
