// MFMA decode attention (decode_attn_mfma.h): further anomalous-channel counts.
#include "decode_attn_mfma.h"

namespace vidkv {

bool launch_attn_mfma_b(const AttnArgs& a, dim3 grid, hipStream_t st) {
  switch (a.n_a) {
    case 24: launch_one<3, true>(a, grid, st); return true;
    case 40: launch_one<5, true>(a, grid, st); return true;
    case 48: launch_one<6, true>(a, grid, st); return true;
    case 56: launch_one<7, true>(a, grid, st); return true;
    case 72: launch_one<9, true>(a, grid, st); return true;
    case 80: launch_one<10, true>(a, grid, st); return true;
    default: return false;
  }
}

}  // namespace vidkv
