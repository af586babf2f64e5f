// Protected-token selection of one sequence by one workgroup of 1024 threads, for sequences short
// enough that a thread keeps its scores in registers (or, from an index list, that the mask fits
// LDS): one launch, or a few workgroups of another launch, instead of a chain of six short ones.
#pragma once
#include "vidkv_common.h"

namespace vidkv {

// Order-preserving map float -> uint32 (ascending).
__device__ __forceinline__ uint32_t fkey(float f) {
  const uint32_t b = __float_as_uint(f + 0.0f);   // -0 and +0 are the same score
  return (b & 0x80000000u) ? ~b : (b | 0x80000000u);
}

constexpr int ONE_THREADS = 1024;
constexpr int ONE_Q = 8;                                  // float4 pieces of scores per thread
constexpr int ONE_MAX_T = ONE_THREADS * 4 * ONE_Q;        // 32768 tokens
constexpr int ONE_COPIES = 32;                            // histogram copies, by lane: one for each bank
constexpr int ONE_BINS = 256;

constexpr int FEW_MAX_GROUPS = 256;                       // of a sequence, where a call has few groups in all

struct OneSelLds {
  int hist[ONE_BINS][ONE_COPIES];                         // index list: the mask (ONE_MAX_T / 32 words)
  int wsum[16], lsum[2][16];
  int pre_s[ONE_Q][16], pre_e[ONE_Q][16];
  int bin, rem;
};

struct OneSelArgs {
  const float* scores;        // [B, T] or NULL
  const int32_t* idx_in;      // [B, n_s] or NULL
  int T, ng, ngc, n_s;
  int32_t* idx;               // IDX, MASK, RANK of the packed buffer
  uint32_t* mask;
  uint32_t* rank;
};

// Inclusive scan over the lanes of a wave, all of them active: inside rows of 16 lanes, then the totals
// of the rows before (register moves: with the exchanges through LDS the selection of 1568 tokens took 10.1 us).
// STEP = 4: v is the same in each four lanes and counts once.
template <int STEP>
__device__ __forceinline__ int wave_scan(int v) {
  if (STEP == 1) {
    v += __builtin_amdgcn_update_dpp(0, v, 0x111, 0xF, 0xF, true);   // from lane - 1
    v += __builtin_amdgcn_update_dpp(0, v, 0x112, 0xF, 0xF, true);   // - 2
  }
  v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xF, 0xF, true);     // - 4
  v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xF, 0xF, true);     // - 8
  v += __builtin_amdgcn_update_dpp(0, v, 0x142, 0xA, 0xF, false);    // rows 1 and 3: lane 15 of the row before
  v += __builtin_amdgcn_update_dpp(0, v, 0x143, 0xC, 0xF, false);    // rows 2 and 3: lane 31
  return v;
}

// Exclusive scan of one int per thread over the 1024 threads.
__device__ __forceinline__ int one_exscan(int v, int* wsum) {
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  const int inc = wave_scan<1>(v);
  __syncthreads();                                        // wsum may still be read
  if (lane == 63) wsum[wv] = inc;
  __syncthreads();
  int base = 0;
#pragma unroll
  for (int i = 0; i < 16; ++i) base += i < wv ? wsum[i] : 0;
  return base + inc - v;
}

// The n_s largest scores (ties: lower index first) by a radix select on the ordered 32-bit keys
// (four digits of 8 bits), then IDX, MASK and RANK in token order.  Thread t holds the scores of the
// pieces q 1024 + t, four tokens each; a wave of a slab q covers 256 consecutive tokens.
// A digit's copies lie in the 32 banks, so that at most two lanes of a wave add to one word, whatever the
// scores are: saliency scores crowd into few digits, and equal, clipped or coarse ones (padding) into one.
// A launch of its own takes 8.8 us at 1568 tokens, 20.9 at 32768 with scattered scores and 19.4 with equal ones.
// (Three digits of 11, 11 and 10 bits, four copies that shared a bank: 8.9, 22.8 and 56; the six-launch
// chain: 22.5, 23.6 and 25.5.)
__device__ __forceinline__ void select_one(const OneSelArgs& a, int b, OneSelLds& s) {
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int np = a.T >> 2, nq = (np + ONE_THREADS - 1) / ONE_THREADS;
  uint32_t key[ONE_Q][4];                                 // of a piece without tokens: never looked at (p < np)
  uint32_t sel[ONE_Q], tie[ONE_Q];                        // bit j: token j of the piece is in / has the last key
  int take_eq = 0;
  if (a.scores) {
    const float4* sc4 = reinterpret_cast<const float4*>(a.scores + (size_t)b * a.T);
    float4 v[ONE_Q];
#pragma unroll
    for (int q = 0; q < ONE_Q; ++q) {
      const int p = q * ONE_THREADS + tid;
      v[q] = p < np ? sc4[p] : float4{0.f, 0.f, 0.f, 0.f};
    }
    // my eight words of the histogram: those of bin 255 - t / 4 (bins descend with t), copies 8 (t % 4) ..
    const int bin = ONE_BINS - 1 - (tid >> 2);
    int4* mine = reinterpret_cast<int4*>(&s.hist[bin][8 * (tid & 3)]);
    mine[0] = mine[1] = int4{0, 0, 0, 0};
    uint32_t prefix = 0, pmask = 0;
    int rem = a.n_s;
    __syncthreads();
#pragma unroll
    for (int q = 0; q < ONE_Q; ++q) {
      key[q][0] = fkey(v[q].x); key[q][1] = fkey(v[q].y); key[q][2] = fkey(v[q].z); key[q][3] = fkey(v[q].w);
    }
#pragma unroll
    for (int level = 0; level < 4; ++level) {
      const int shift = 24 - 8 * level;
#pragma unroll
      for (int q = 0; q < ONE_Q; ++q)
        if (q * ONE_THREADS + tid < np) {
#pragma unroll
          for (int j = 0; j < 4; ++j)
            if ((key[q][j] & pmask) == prefix)
              atomicAdd(&s.hist[(key[q][j] >> shift) & (ONE_BINS - 1)][lane & (ONE_COPIES - 1)], 1);
        }
      __syncthreads();
      // the bin's count, its words cleared for the next level; then the keys in higher bins
      const int4 x = mine[0], y = mine[1];
      mine[0] = mine[1] = int4{0, 0, 0, 0};
      int c = x.x + x.y + x.z + x.w + y.x + y.y + y.z + y.w;
      c += __builtin_amdgcn_update_dpp(0, c, 0xB1, 0xF, 0xF, true);   // the lane beside
      c += __builtin_amdgcn_update_dpp(0, c, 0x4E, 0xF, 0xF, true);   // the pair beside
      const int inc = wave_scan<4>(c);                    // over the 16 bins of my wave, 4 lanes each
      if (lane == 63) s.lsum[level & 1][wave] = inc;
      __syncthreads();
      int above = inc - c;
#pragma unroll
      for (int i = 0; i < 16; ++i) above += i < wave ? s.lsum[level & 1][i] : 0;
      if ((tid & 3) == 0 && above < rem && rem <= above + c) {   // exactly one thread
        s.bin = bin;
        s.rem = rem - above;
      }
      __syncthreads();
      prefix |= (uint32_t)s.bin << shift;
      pmask |= (uint32_t)(ONE_BINS - 1) << shift;
      rem = s.rem;
    }
    take_eq = rem;
#pragma unroll
    for (int q = 0; q < ONE_Q; ++q) {
      sel[q] = tie[q] = 0;
      if (q * ONE_THREADS + tid < np) {
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          sel[q] |= (key[q][j] > prefix ? 1u : 0u) << j;
          tie[q] |= (key[q][j] == prefix ? 1u : 0u) << j;
        }
      }
    }
  } else {
    uint32_t* m = reinterpret_cast<uint32_t*>(&s.hist[0][0]);
    if (tid < ONE_MAX_T / 32) m[tid] = 0;
    __syncthreads();
    for (int i = tid; i < a.n_s; i += ONE_THREADS) {
      const int t = a.idx_in[(size_t)b * a.n_s + i];
      if (t >= 0 && t < a.T) atomicOr(&m[t >> 5], 1u << (t & 31));   // an index outside the cache is ignored
    }
    for (int g = a.ng + tid; g < a.ngc; g += ONE_THREADS) a.mask[(size_t)b * a.ngc + g] = 0;   // room behind the tokens
    __syncthreads();
#pragma unroll
    for (int q = 0; q < ONE_Q; ++q) {
      const int p = q * ONE_THREADS + tid;                // < ONE_MAX_T / 4: inside the mask
      sel[q] = (m[p >> 3] >> (4 * (p & 7))) & 15u;
      tie[q] = 0;
    }
  }
  // counts per (slab, wave), in token order; then the sums of all before each
#pragma unroll
  for (int q = 0; q < ONE_Q; ++q) {
    int cs = 0, ce = 0;
    if (q < nq) {
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        cs += __popcll(__ballot((sel[q] >> j) & 1u));
        ce += __popcll(__ballot((tie[q] >> j) & 1u));
      }
    }
    if (lane == 0) { s.pre_s[q][wave] = cs; s.pre_e[q][wave] = ce; }
  }
  __syncthreads();
  {
    const int cs = tid < ONE_Q * 16 ? s.pre_s[0][tid] : 0, ce = tid < ONE_Q * 16 ? s.pre_e[0][tid] : 0;
    const int ps = one_exscan(cs, s.wsum);
    const int pe = one_exscan(ce, s.wsum);
    if (tid < ONE_Q * 16) { s.pre_s[0][tid] = ps; s.pre_e[0][tid] = pe; }
  }
  __syncthreads();
#pragma unroll
  for (int q = 0; q < ONE_Q; ++q) {
    if (q >= nq) break;
    const int p = q * ONE_THREADS + tid;
    int bs = s.pre_s[q][wave], be = s.pre_e[q][wave];     // selected / tied tokens before mine
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const unsigned long long ms = __ballot((sel[q] >> j) & 1u), me = __ballot((tie[q] >> j) & 1u);
      bs += __builtin_amdgcn_mbcnt_hi((uint32_t)(ms >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)ms, 0u));
      be += __builtin_amdgcn_mbcnt_hi((uint32_t)(me >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)me, 0u));
    }
    const int first = bs + min(be, take_eq);              // protected tokens before my first
    uint32_t in = 0;
    int r = first;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const bool t = (tie[q] >> j) & 1u;
      if (((sel[q] >> j) & 1u) || (t && be < take_eq)) {
        in |= 1u << j;
        if (r < a.n_s) a.idx[(size_t)b * a.n_s + r] = 4 * p + j;
        ++r;
      }
      be += t ? 1 : 0;
    }
    uint32_t w = in << (4 * (lane & 7));                  // 8 lanes: one group
    w |= __shfl_xor(w, 1, 64);
    w |= __shfl_xor(w, 2, 64);
    w |= __shfl_xor(w, 4, 64);
    if ((lane & 7) == 0 && (p >> 3) < a.ng) {
      a.mask[(size_t)b * a.ngc + (p >> 3)] = w;
      a.rank[(size_t)b * a.ngc + (p >> 3)] = (uint32_t)first;
    }
  }
}

// The same for few groups, one workgroup of 1024 threads each: the rank of every token of group g by counting, 32 tokens
// against 32 parts of the keys.  Only MASK is written; RANK and IDX come with the value coding.  Quadratic, but spread over as
// many workgroups as there are groups, and one pass instead of four digits' and their barriers by a single one:
// (1568 tokens: the launch with the range pass of one head 9.0 us with select_one, 4.1 so.)
struct FewSelLds {
  u32x4 key[FEW_MAX_GROUPS * 8];
  int cnt[16][32];
};

__device__ __forceinline__ void few_select(const OneSelArgs& a, int b, int g, FewSelLds& s) {
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int np = a.T >> 2;
  const float4* sc4 = reinterpret_cast<const float4*>(a.scores + (size_t)b * a.T);
  for (int p = tid; p < np; p += ONE_THREADS) {
    const float4 v = sc4[p];
    s.key[p] = u32x4{fkey(v.x), fkey(v.y), fkey(v.z), fkey(v.w)};
  }
  __syncthreads();
  const int t = 32 * g + (lane & 31), part = 2 * wave + (lane >> 5), at = g >> 2;
  const uint32_t k = reinterpret_cast<const uint32_t*>(&s.key[0])[t];
  // tokens before mine that have my key or a larger one, tokens behind it that have a larger one.  Of pieces part + 32 i
  // those with i < at lie before the group, those with i > at behind it
  int c = 0;
  for (int i = 0; i < at; ++i) {
    const u32x4 v = s.key[part + 32 * i];
#pragma unroll
    for (int e = 0; e < 4; ++e) c += v[e] >= k ? 1 : 0;
  }
  if (part + 32 * at < np) {
    const u32x4 v = s.key[part + 32 * at];
#pragma unroll
    for (int e = 0; e < 4; ++e) c += v[e] > k || (v[e] == k && 4 * (part + 32 * at) + e < t) ? 1 : 0;
  }
  for (int p = part + 32 * (at + 1); p < np; p += 32) {
    const u32x4 v = s.key[p];
#pragma unroll
    for (int e = 0; e < 4; ++e) c += v[e] > k ? 1 : 0;
  }
  c += __shfl_xor(c, 32, 64);
  if (lane < 32) s.cnt[wave][lane] = c;
  __syncthreads();
  if (wave == 0) {
    int r = 0;
#pragma unroll
    for (int i = 0; i < 16; ++i) r += s.cnt[i][lane & 31];
    const uint32_t w = (uint32_t)__ballot(r < a.n_s);
    if (lane == 0) a.mask[(size_t)b * a.ngc + g] = w;
  }
}

// MASK of sequence b from its index list (an index outside the cache is ignored), 0 in the room behind the tokens.
__device__ __forceinline__ void few_list(const OneSelArgs& a, int b, FewSelLds& s) {
  uint32_t* m = reinterpret_cast<uint32_t*>(&s.key[0]);
  const int tid = threadIdx.x;
  if (tid < FEW_MAX_GROUPS) m[tid] = 0;
  __syncthreads();
  for (int i = tid; i < a.n_s; i += ONE_THREADS) {
    const int t = a.idx_in[(size_t)b * a.n_s + i];
    if (t >= 0 && t < a.T) atomicOr(&m[t >> 5], 1u << (t & 31));
  }
  __syncthreads();
  for (int g = tid; g < a.ngc; g += ONE_THREADS) a.mask[(size_t)b * a.ngc + g] = g < a.ng ? m[g] : 0u;
}

OneSelArgs one_sel_args(const Geom& g, const float* scores, const int32_t* idx, uint8_t* packed);

}  // namespace vidkv
