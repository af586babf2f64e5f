// MFMA decode attention (decode_attn_mfma.h): further anomalous-channel counts.
#include "decode_attn_mfma.h"

namespace vidkv {

bool launch_attn_mfma_c(const AttnArgs& a, dim3 grid, hipStream_t st) {
  switch (a.n_a) {
    case 88: launch_one<11, true>(a, grid, st); return true;
    case 104: launch_one<13, true>(a, grid, st); return true;
    case 112: launch_one<14, true>(a, grid, st); return true;
    case 120: launch_one<15, true>(a, grid, st); return true;
    case 128: launch_one<16, true>(a, grid, st); return true;
    default: return false;
  }
}

}  // namespace vidkv
