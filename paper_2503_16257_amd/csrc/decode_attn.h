// Shared declarations of the decode-attention kernels.
#pragma once
#include "mfma_util.h"

namespace vidkv {

struct AttnArgs {
  const _Float16* q;         // [B, Hq, 128]
  const uint8_t* kperm;      // key PERM section (whole buffer)
  const uint8_t* krec;       // key REC section (whole buffer)
  const uint8_t* vrec;       // value REC section (whole buffer)
  const uint32_t* vmask;     // [B, ngc] or unused
  const uint32_t* vrank;     // [B, ngc]
  const _Float16* vrows;     // protected rows: [L, B, H, n_s, 128] fp16, or 2-bit records
                             // [L, B, H, npg] of PREC bytes when sal_bits == 2
  const _Float16* ktail;     // [B, H, cap, 128]
  const _Float16* vtail;
  const int32_t* tail_len;   // [B] or NULL
  // one partial per (split, sequence, query head): o[128], and m, l with
  // p = 2^(score2 - m), l = sum p, o = sum p v
  float* part_o;             // [nsplit + tail splits, B, Hq, 128]
  float* part_ml;            // [nsplit + tail splits, B, Hq, 2]
  int layer, B, H, Hq, rep, ng, n_a, n_n, n_s, krec_bytes, cap, nsplit, gps;
  int ngc;                   // groups of capacity: stride of the per-head record arrays
  int use_fft;               // normal key channels coded by Eq. 5 (1) or by Eq. 4 at 1 bit (0)
  int sal_bits, npg;         // protected rows kept as fp16 (16) or Eq. 4 codes (2); groups of 32 rows
  int tail_per;              // 32-token steps of the residual buffer per tail split
  float scale2;              // softmax scale * log2(e): scores live in the exp2 domain
};

// the packed tokens; one instantiation per anomalous-channel count (any multiple of 8 up to 128)
void launch_attn_mfma(const AttnArgs& a, dim3 grid, hipStream_t st);

}  // namespace vidkv
