// MFMA decode attention (decode_attn_mfma.h): the counts of decode_attn_mfma.hip with
// workgroups for the residual tokens in the same grid.
#include "decode_attn_mfma.h"

namespace vidkv {

bool launch_attn_mfma_t(const AttnArgs& a, dim3 grid, hipStream_t st) {
  switch (a.n_a) {
    case 0: launch_one<0, true>(a, grid, st); return true;
    case 8: launch_one<1, true>(a, grid, st); return true;
    case 16: launch_one<2, true>(a, grid, st); return true;
    case 32: launch_one<4, true>(a, grid, st); return true;
    case 64: launch_one<8, true>(a, grid, st); return true;
    case 96: launch_one<12, true>(a, grid, st); return true;
    default: return false;
  }
}

}  // namespace vidkv
