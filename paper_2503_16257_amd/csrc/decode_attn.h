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

__device__ __forceinline__ float swap_sum32(float v) {       // v(lane) + v(lane ^ 32)
  auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}
__device__ __forceinline__ float swap_sum16(float v) {       // v(lane) + v(lane ^ 16)
  auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}
__device__ __forceinline__ float swap_max32(float v) {
  auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
__device__ __forceinline__ float swap_max16(float v) {
  auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}

// What the four waves of a workgroup leave for its partial: sums in ow (a wave's [8 heads][128 channels]), maxima and
// denominators in mw, lw, [head][wave].
//
// A wave's running sums o[m][i] - row 4 kb + i of the score tile's columns, (half, head), channel 16 m + x16 - into ow:
// the rows of the second half of a head live 32 lanes away from those of its first.  One lane-half swap of the
// register pair (tile m, tile m + 4) and one addition leave the sums of tile m in lanes 0..31 and those of tile m + 4
// in lanes 32..63.
__device__ __forceinline__ void put_wave_sums(const f4 (&o)[8], float* ow, int x16, int kb) {
#pragma unroll
  for (int m = 0; m < 4; ++m)
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(o[m][i]), __float_as_uint(o[m + 4][i]), false, false);
      const float s = __uint_as_float(r[0]) + __uint_as_float(r[1]);
      ow[(4 * (kb & 1) + i) * D + 16 * (m + 4 * (kb >> 1)) + x16] = s;
    }
}
// The workgroup's partial: four channels of one head a thread, everything read at once (one channel of four heads one
// after another, each behind the reads of the maxima: 1.2 to 1.5 us; now 0.4).  ow, wave_stride: in bytes.
__device__ __forceinline__ void put_partial(const AttnArgs& a, int split, int kvh, int b, int tid, const float (&mw)[8][4],
                                            const float (&lw)[8][4], const uint8_t* ow, int wave_stride) {
  const int h = tid >> 5, c4 = tid & 31;
  const f4 m4 = *reinterpret_cast<const f4*>(&mw[h][0]), l4 = *reinterpret_cast<const f4*>(&lw[h][0]);
  f4 x[4];
#pragma unroll
  for (int w = 0; w < 4; ++w) x[w] = *reinterpret_cast<const f4*>(ow + w * wave_stride + (h * D + 4 * c4) * sizeof(float));
  const float M = fmaxf(fmaxf(m4[0], m4[1]), fmaxf(m4[2], m4[3]));
  f4 acc = f4{0.f, 0.f, 0.f, 0.f};
  float L = 0.0f;
#pragma unroll
  for (int w = 0; w < 4; ++w) {
    const bool any = m4[w] != -INFINITY;                      // an empty wave's sums are never looked at
    const float f = any ? __builtin_amdgcn_exp2f(m4[w] - M) : 0.0f;
    L += any ? f * l4[w] : 0.0f;
#pragma unroll
    for (int i = 0; i < 4; ++i) acc[i] += any ? f * x[w][i] : 0.0f;
  }
  if (h < a.rep) {
    const long long row = ((long long)split * a.B + b) * a.Hq + kvh * a.rep + h;
    *reinterpret_cast<f4*>(a.part_o + row * D + 4 * c4) = acc;
    if (c4 == 0) *reinterpret_cast<float2*>(a.part_ml + row * 2) = float2{M, L};
  }
}

typedef _Float16 h4 __attribute__((ext_vector_type(4)));
typedef short s16x4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ h2 rtz2(float a, float b) { return __builtin_bit_cast(h2, __builtin_amdgcn_cvt_pkrtz(a, b)); }

struct alignas(256) TailLds {
  uint8_t v[4][32 * 2 * D];               // per wave: a block's value rows, swizzled; then the wave's sums
  float mw[8][4], lw[8][4];               // [head][wave]
};

// The fp16 residual tokens (Alg. 1's X_Kr, X_Vr): one workgroup = one (tail split, KV head,
// sequence); split ts takes the 32-token blocks ts * tail_per .. of the buffer, its waves in turn, and writes its
// partial (o, m, l) as split index nsplit + ts.  Bound by the memory where there are many of them, by one chain of
// latencies where there are few.  Both contractions run on the matrix cores, K rows straight from memory as
// operands, value rows through LDS and its transposing reads; everything a block needs is asked for at once.
// As exact as in 32-bit arithmetic.  q, keys and values are fp16 numbers with exact products.  A probability enters as four
// fp16 numbers that add up to it, each cut off behind 11 bits, in the rows of the 8 heads and the 8 that would be empty
// of two products a tile: all its 24 bits down to 2^-48 of the running maximum, what is above 2^-72 below it.  (A product takes a
// subnormal operand for one of 2^-14 where it aligns its sum, and cuts off 24 bits below: 2^-53 of the running maximum times a
// value here, less than 2^-25 in a result of up to 4096 tokens; of keys, queries and values that are all a few 2^-24, 2^-17 of a sum.)
__device__ __forceinline__ void attn_tail_part(const AttnArgs& a, int ts, int kvh, int b, TailLds& t) {
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int x16 = lane & 15, kb = lane >> 4, hcol = x16 & 7, R = a.rep;
  const f4 zero = f4{0.f, 0.f, 0.f, 0.f};
  int tl = a.tail_len ? a.tail_len[b] : 0;
  tl = min(max(tl, 0), a.cap);
  const int it0 = ts * a.tail_per + wave, it1 = min((tl + 31) / 32, (ts + 1) * a.tail_per);
  const long long head_row0 = ((long long)b * a.H + kvh) * a.cap;
  f4 o[8];
#pragma unroll
  for (int m = 0; m < 8; ++m) o[m] = zero;
  float m_run = -INFINITY, l_run = 0.0f;
  if (it0 < it1) {
    Op Bq[4];                                        // q of my column's head at channels 32 u + 8 kb + e
    const u32x4* q4 = reinterpret_cast<const u32x4*>(a.q + ((long long)b * a.Hq + kvh * R + (hcol < R ? hcol : 0)) * D) + kb;
#pragma unroll
    for (int u = 0; u < 4; ++u) Bq[u].q = q4[4 * u];
    uint8_t* vrow = &t.v[wave][0];
    // a transposing read hands lane x16 of kb the rows 4 kb .. 4 kb + 3 (of either half) of channel 16 m + x16
    const int rr = 4 * kb + (x16 >> 2);
    const uint32_t at = (uint32_t)reinterpret_cast<uintptr_t>(vrow) + rr * 2 * D + (rr & 7) * 32 + (x16 & 3) * 8;
    // part k is taken times 2^(15 + 11 k), all below 2^15 but p = 1: parts 0 and 2 in rows 0..7, 1 and 3 in rows 8..15
    const bool odd = x16 >= 8;
    const float skip = odd ? -1.0f : 0.0f, up = odd ? 0x1p11f : 1.0f;
    for (int it = it0; it < it1; it += 4) {
      const int tok0 = it * 32, nt = min(32, tl - tok0);
      // (a row past the end repeats the last one and counts 0 times)
      const u32x4* kt = reinterpret_cast<const u32x4*>(a.ktail + (head_row0 + tok0) * D);
      const u32x4* vt = reinterpret_cast<const u32x4*>(a.vtail + (head_row0 + tok0) * D);
      Op Ak[2][4];
      u32x4 vv[8];
#pragma unroll
      for (int mt = 0; mt < 2; ++mt)
#pragma unroll
        for (int u = 0; u < 4; ++u) Ak[mt][u].q = kt[min(16 * mt + x16, nt - 1) * 16 + 4 * u + kb];
#pragma unroll
      for (int j = 0; j < 8; ++j) vv[j] = vt[min(4 * j + kb, nt - 1) * 16 + x16];
      __builtin_amdgcn_sched_barrier(0);
      f4 S[2] = {zero, zero};
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        S[0] = mma(Ak[0][u], Bq[u], S[0]);
        S[1] = mma(Ak[1][u], Bq[u], S[1]);
      }
      // row r keeps its 16-byte pieces in the order piece ^ 2 (r & 7), so that the transposing reads spread over the banks
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        const int r = 4 * j + kb;
        *reinterpret_cast<u32x4*>(vrow + r * 2 * D + ((x16 ^ (2 * (r & 7))) * 16)) = vv[j];
      }
      asm volatile("" ::: "memory");
      // softmax in the exp2 domain: my column at tokens 4 kb + i (i < 4) and 16 + 4 kb + i - 4
      float sc[8];
#pragma unroll
      for (int i = 0; i < 8; ++i) sc[i] = slot_token(kb, i) < nt ? S[i >> 2][i & 3] * a.scale2 : -INFINITY;
      const float mx = fmaxf(fmaxf(fmaxf(sc[0], sc[1]), fmaxf(sc[2], sc[3])), fmaxf(fmaxf(sc[4], sc[5]), fmaxf(sc[6], sc[7])));
      const float m_new = fmaxf(m_run, swap_max16(swap_max32(mx)));
      const float al = m_run == -INFINITY ? 0.0f : __builtin_amdgcn_exp2f(m_run - m_new);
      l_run *= al;
      m_run = m_new;
      Op A[2];
#pragma unroll
      for (int i = 0; i < 8; i += 2) {
        float p[2];
#pragma unroll
        for (int e = 0; e < 2; ++e) {
          p[e] = sc[i + e] == -INFINITY ? 0.0f : __builtin_amdgcn_exp2f(sc[i + e] - m_new);
          l_run += p[e];
          p[e] *= 0x1p15f;
        }
        // p: what is left behind a part, at the next one's scale.  Behind the one in front of mine (none for part 0), mine,
        // the next one, and mine again
        auto behind = [&](h2 part, float take, float scale) {
#pragma unroll
          for (int e = 0; e < 2; ++e) p[e] = fmaf((float)part[e], take, p[e]) * scale;
        };
        behind(rtz2(p[0], p[1]), skip, up);
        A[0].p[i / 2] = rtz2(p[0], p[1]);
        behind(A[0].p[i / 2], -1.0f, 0x1p11f);
        behind(rtz2(p[0], p[1]), -1.0f, 0x1p11f);
        A[1].p[i / 2] = rtz2(p[0], p[1]);
      }
      if (it != it0) {
        // the sums are laid out by score-tile column as ROW 4 kb + i
        float ar[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) ar[i] = __shfl(al, 4 * kb + i, 64);
#pragma unroll
        for (int m = 0; m < 8; ++m)
#pragma unroll
          for (int i = 0; i < 4; ++i) o[m][i] *= ar[i];
      }
      s16x4 lo4[8], hi4[8];                          // all requested before the first is used
#pragma unroll
      for (int m = 0; m < 8; ++m) {
        lo4[m] = __builtin_amdgcn_ds_read_tr16_b64_v4i16(reinterpret_cast<__attribute__((address_space(3))) s16x4*>(at ^ (m * 32)));
        hi4[m] = __builtin_amdgcn_ds_read_tr16_b64_v4i16(reinterpret_cast<__attribute__((address_space(3))) s16x4*>((at + 16 * 2 * D) ^ (m * 32)));
      }
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int m = 0; m < 8; ++m) {
        Op B;
        *reinterpret_cast<s16x4*>(&B.u[0]) = lo4[m];
        *reinterpret_cast<s16x4*>(&B.u[2]) = hi4[m];
        const f4 C = mma(A[1], B, zero);
        o[m] = mma(A[0], B, o[m]);
#pragma unroll
        for (int i = 0; i < 4; ++i) o[m][i] = fmaf(0x1p-22f, C[i], o[m][i]);
      }
      asm volatile("" ::: "memory");
    }
    l_run = swap_sum16(swap_sum32(l_run));
    const float row = (kb >> 1) ? 0x1p-26f : 0x1p-15f;       // of my rows' part
#pragma unroll
    for (int m = 0; m < 8; ++m) o[m] *= row;
  }
  put_wave_sums(o, reinterpret_cast<float*>(&t.v[wave][0]), x16, kb);
  if (kb == 0 && x16 < 8) { t.mw[hcol][wave] = m_run; t.lw[hcol][wave] = l_run; }
  __syncthreads();
  put_partial(a, a.nsplit + ts, kvh, b, tid, t.mw, t.lw, &t.v[0][0], 32 * 2 * D);
}

// The packed tokens, and with a grid.x beyond a.nsplit the residual tokens; one instantiation per
// anomalous-channel count (any multiple of 8 up to 128).
void launch_attn_mfma(const AttnArgs& a, dim3 grid, hipStream_t st);

}  // namespace vidkv
