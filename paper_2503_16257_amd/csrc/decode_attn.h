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
  int layer, B, H, Hq, rep, ng, n_a, n_s, cap, nsplit, gps;
  int ngc;                   // groups of capacity: stride of the per-head record arrays
  int use_fft;               // normal key channels coded by Eq. 5 (1) or by Eq. 4 at 1 bit (0)
  int sal_bits, npg;         // protected rows kept as fp16 (16) or Eq. 4 codes (2); groups of 32 rows
  int early;                 // at most one workgroup per compute unit: the first pair's values are requested at the start
  int tail_per;              // 32-token steps of the residual buffer per tail split
  float scale2;              // softmax scale * log2(e): scores live in the exp2 domain
};

struct alignas(16) TailLds {              // (16: q and P are read four at a time)
  float q[MAX_REP][D];
  float P[MAX_REP][32];
  float alpha[MAX_REP];
};

// The fp16 residual tokens (Alg. 1's X_Kr, X_Vr): one workgroup = one (tail split, KV head,
// sequence); split ts takes the 32-token steps ts * tail_per .. of the buffer and writes its
// partial (o, m, l) as split index nsplit + ts.  Thread roles: scores (token = tid % 32,
// head = tid / 32), output (channel = tid % 128, heads tid / 128 + 2 i).
__device__ __forceinline__ void attn_tail_part(const AttnArgs& a, int ts, int kvh, int b, TailLds& t) {
  const int split = a.nsplit + ts;
  const int tid = threadIdx.x;
  const int R = a.rep;
  float (&t_q)[MAX_REP][D] = t.q;
  float (&t_P)[MAX_REP][32] = t.P;
  float (&t_alpha)[MAX_REP] = t.alpha;
  for (int i = tid; i < R * D; i += 256)
    t_q[i >> 7][i & 127] = (float)a.q[((long long)b * a.Hq + kvh * R + (i >> 7)) * D + (i & 127)];
  const int t_s = tid & 31, h_s = tid >> 5;
  const int c_o = tid & 127, half_o = tid >> 7;
  float m_run = -INFINITY, l_run = 0.0f;
  float acc[4] = {0.f, 0.f, 0.f, 0.f};
  int tl = a.tail_len ? a.tail_len[b] : 0;
  tl = min(max(tl, 0), a.cap);
  const int it0 = ts * a.tail_per;
  const int n_iter = max(0, min((tl + 31) / 32, it0 + a.tail_per) - it0);
  const long long head_row0 = ((long long)b * a.H + kvh) * a.cap;
  for (int it = 0; it < n_iter; ++it) {
    const int tok0 = (it0 + it) * 32;
    const int nt = min(32, tl - tok0);
    // everything this step reads is requested up front: my key row (16 pieces) and my
    // channel of the 32 value rows (a row past the end repeats the last one and is not used)
    const bool scorer = h_s < R && t_s < nt;
    U4H kr[16];
    if (scorer) {
      const u32x4* row = reinterpret_cast<const u32x4*>(a.ktail + (head_row0 + tok0 + t_s) * D);
#pragma unroll
      for (int i = 0; i < 16; ++i) kr[i].u = row[i];
    }
    const _Float16* vcol = a.vtail + (head_row0 + tok0) * D + c_o;
    _Float16 vv[32];
#pragma unroll
    for (int u = 0; u < 32; ++u) vv[u] = vcol[(long long)min(u, nt - 1) * D];
    if (it == 0) __syncthreads();                    // q is in LDS (its loads overlapped the above)
    float score = -INFINITY;
    if (scorer) {
      float v = 0.0f;
#pragma unroll
      for (int i = 0; i < 16; ++i)
#pragma unroll
        for (int e = 0; e < 8; ++e) v += t_q[h_s][i * 8 + e] * (float)kr[i].e[e];
      score = v * a.scale2;
    }
    if (h_s < R) {                                   // online softmax of this step (exp2 domain)
      float mx = score;
#pragma unroll
      for (int d = 16; d >= 1; d >>= 1) mx = fmaxf(mx, __shfl_xor(mx, d, 32));
      const float m_new = fmaxf(m_run, mx);
      const float p = (score == -INFINITY) ? 0.0f : exp2f(score - m_new);
      const float al = (m_run == -INFINITY) ? 0.0f : exp2f(m_run - m_new);
      float ps = p;
#pragma unroll
      for (int d = 16; d >= 1; d >>= 1) ps += __shfl_xor(ps, d, 32);
      l_run = l_run * al + ps;
      m_run = m_new;
      t_P[h_s][t_s] = p;
      if (t_s == 0) t_alpha[h_s] = al;
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int h = half_o + 2 * i;
      if (h < R) {
        float s_acc = acc[i] * t_alpha[h];
#pragma unroll
        for (int u = 0; u < 32; ++u) s_acc += t_P[h][u] * (float)vv[u];   // t_P is 0 past the end
        acc[i] = s_acc;
      }
    }
    __syncthreads();
  }
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int h = half_o + 2 * i;
    if (h < R) a.part_o[(((long long)split * a.B + b) * a.Hq + kvh * R + h) * D + c_o] = acc[i];
  }
  if (h_s < R && t_s == 0) {
    float* ml = a.part_ml + (((long long)split * a.B + b) * a.Hq + kvh * R + h_s) * 2;
    ml[0] = m_run;
    ml[1] = l_run;
  }
}

// The packed tokens, and with a grid.x beyond a.nsplit the residual tokens; one instantiation per
// anomalous-channel count (any multiple of 8 up to 128).
void launch_attn_mfma(const AttnArgs& a, dim3 grid, hipStream_t st);

}  // namespace vidkv
