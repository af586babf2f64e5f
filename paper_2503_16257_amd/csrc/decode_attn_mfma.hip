// MFMA decode attention (decode_attn_mfma.h): the anomalous-channel counts of the workloads,
// and the choice of the instantiation.  Every multiple of 8 up to 128 has one; they are spread
// over four files so that they compile side by side.  (A scalar kernel served the counts outside
// 0, 8, 16, 32, 64, 128 before: 20.4 us at n_a = 96, 2 sequences of 3136 tokens, 4 KV heads; a
// 28-layer decode step of that shape went from 698 to 569 us with this kernel, whose other
// launches and host work are the rest.)
#include "decode_attn_mfma.h"

namespace vidkv {

bool launch_attn_mfma_t(const AttnArgs& a, dim3 grid, hipStream_t st);
bool launch_attn_mfma_b(const AttnArgs& a, dim3 grid, hipStream_t st);
bool launch_attn_mfma_c(const AttnArgs& a, dim3 grid, hipStream_t st);

void launch_attn_mfma(const AttnArgs& a, dim3 grid, hipStream_t st) {
  if ((int)grid.x > a.nsplit && launch_attn_mfma_t(a, grid, st)) return;
  switch (a.n_a) {
    case 0:   launch_one<0, false>(a, grid, st); break;
    case 8:   launch_one<1, false>(a, grid, st); break;
    case 16:  launch_one<2, false>(a, grid, st); break;
    case 32:  launch_one<4, false>(a, grid, st); break;
    case 64:  launch_one<8, false>(a, grid, st); break;
    case 96:  launch_one<12, false>(a, grid, st); break;
    default:
      if (!launch_attn_mfma_b(a, grid, st)) launch_attn_mfma_c(a, grid, st);
  }
}

}  // namespace vidkv
