// Protected value rows at 2 bits (Alg. 2, STPQuant), as a piece that a launch of its own or a part
// of another one runs.
#pragma once
#include "select_values.h"

namespace vidkv {

// Alg. 2, STPQuant, protected branch: the protected rows of one head, gathered
// in token order, coded with Eq. 4 at 2 bits per channel over groups of 32
// protected tokens (the last group may hold fewer).  One wave codes one record, lane = two adjacent
// channels: a row is one 256-byte request of the wave, all 32 rows are requested at once, and the
// codes of a lane pair make the record's bytes.  (A thread per channel, 2-byte loads: 11.9 us for 4480
// records of the 28 x 6272 token cache.  Behind the key coding pass's workgroups, in the same launch,
// the whole call took 116.5 us; in front of them 119; as launches of their own one gap more.)  Record: codes [32 rows][32 bytes] (channel
// 4 j + r of a row in bits 2r.. of byte j), fp16 s[128], fp16 z[128].
struct Protect2Args {
  const _Float16* V;
  int T, B, H, n_s, npg;
  const int32_t* idx;
  uint8_t* out;
  long long total;            // records
  const uint32_t* mask;       // where IDX is not there yet
  int ngc;
};

typedef u32x4 Protect2Lds[64];       // the 1024 bytes of codes of a wave's record

// FROM_MASK (up to FEW_MAX_GROUPS groups a sequence): the record's tokens are found in MASK.
template <bool FROM_MASK = false>
__device__ __forceinline__ void protect2_part(const Protect2Args& a, long long rec_id, Protect2Lds& lds) {
  const int lane = threadIdx.x & 63;
  const long long hd = rec_id / a.npg;
  const int pg = (int)(rec_id - hd * a.npg);
  const int b = (int)((hd / a.H) % a.B);
  const int cnt = min(G, a.n_s - pg * G);
  int32_t* found = reinterpret_cast<int32_t*>(&lds[0]);
  if (FROM_MASK) {
    constexpr int W = FEW_MAX_GROUPS / 64;             // my words: W lane ..
    const uint32_t* mk = a.mask + (size_t)b * a.ngc;
    const int ng = a.T / G;
    uint32_t w[W];
    int c = 0;
#pragma unroll
    for (int i = 0; i < W; ++i) w[i] = mk[min(W * lane + i, ng - 1)];
#pragma unroll
    for (int i = 0; i < W; ++i) {
      if (W * lane + i >= ng) w[i] = 0u;
      c += __popc(w[i]);
    }
    int r = wave_scan<1>(c) - c - pg * G;              // rank of my first protected token inside the record
    if (lane < G) found[lane] = a.T;                   // (a list with repeats has fewer tokens: clamped below)
    asm volatile("" ::: "memory");
#pragma unroll
    for (int i = 0; i < W; ++i) {
      uint32_t m = r + __popc(w[i]) > 0 && r < G ? w[i] : 0u;
      int at = r;
      while (m) {
        const int t = __ffs(m) - 1;
        m &= m - 1;
        if (at >= 0 && at < G) found[at] = (W * lane + i) * G + t;
        ++at;
      }
      r += __popc(w[i]);
    }
    asm volatile("" ::: "memory");
  }
  // rows beyond the last one repeat it: every load is valid and changes neither min nor max
  // (an index list with repeated or out-of-range entries leaves the end of IDX unwritten:
  // whatever is there is clamped into the tensor, such rows are never read back)
  const int last = min(lane & 31, cnt - 1);
  const int tok = min(max(FROM_MASK ? found[last] : a.idx[(size_t)b * a.n_s + pg * G + last], 0), a.T - 1);
  const uint32_t* head = reinterpret_cast<const uint32_t*>(a.V + hd * (long long)a.T * D) + lane;
  uint32_t xr[G];
#pragma unroll
  for (int r = 0; r < G; ++r) xr[r] = head[(size_t)__builtin_amdgcn_readlane(tok, r) * (D / 2)];
  float lo[2] = {65504.0f, 65504.0f}, hi[2] = {-65504.0f, -65504.0f};
#pragma unroll
  for (int r = 0; r < G; ++r) {
    const h2 x = __builtin_bit_cast(h2, xr[r]);
#pragma unroll
    for (int e = 0; e < 2; ++e) {
      lo[e] = fminf(lo[e], (float)x[e]);
      hi[e] = fmaxf(hi[e], (float)x[e]);
    }
  }
  float rng[2], inv[2];
#pragma unroll
  for (int e = 0; e < 2; ++e) {
    rng[e] = hi[e] - lo[e];
    inv[e] = rng[e] > 0.0f ? 3.0f / rng[e] : 0.0f;
  }
  uint32_t w[4] = {0u, 0u, 0u, 0u};          // my two channels' codes, 4 bits a row
#pragma unroll
  for (int r = 0; r < G; ++r) {
    const h2 x = __builtin_bit_cast(h2, xr[r]);
    uint32_t nib = 0;
#pragma unroll
    for (int e = 0; e < 2; ++e) {
      float u = ((float)x[e] - lo[e]) * inv[e];
      u = fminf(fmaxf(rintf(u), 0.0f), 3.0f);
      nib |= (uint32_t)u << (2 * e);
    }
    w[r >> 3] |= (r < cnt ? nib : 0u) << (4 * (r & 7));
  }
  // lane pair: the even lane writes the bytes of rows 0-15, the odd one those of rows 16-31
  uint8_t* by = reinterpret_cast<uint8_t*>(&lds[0]);
  const int odd = lane & 1;
#pragma unroll
  for (int k = 0; k < 2; ++k) {
    const uint32_t mine = odd ? w[2 + k] : w[k], theirs = __shfl_xor(odd ? w[k] : w[2 + k], 1, 64);
    const uint32_t l4 = odd ? theirs : mine, h4 = odd ? mine : theirs;
#pragma unroll
    for (int i = 0; i < 8; ++i)
      by[(16 * odd + 8 * k + i) * 32 + (lane >> 1)] = (uint8_t)(((l4 >> (4 * i)) & 15u) | (((h4 >> (4 * i)) & 15u) << 4));
  }
  uint8_t* rec = a.out + (hd * a.npg + pg) * (long long)PREC;
  const h2 s16 = h2{(_Float16)(rng[0] / 3.0f), (_Float16)(rng[1] / 3.0f)}, z16 = h2{(_Float16)lo[0], (_Float16)lo[1]};
  reinterpret_cast<uint32_t*>(rec + 1024)[lane] = __builtin_bit_cast(uint32_t, s16);
  reinterpret_cast<uint32_t*>(rec + 1280)[lane] = __builtin_bit_cast(uint32_t, z16);
  reinterpret_cast<u32x4*>(rec)[lane] = lds[lane];       // same wave: its LDS writes are in order before the read
}

Protect2Args protect2_args(const Geom& g, const void* V, uint8_t* packed);

}  // namespace vidkv
