// Per-channel range over all tokens and top-n_a channel selection of the key quantizer (Alg. 3), as
// pieces that a launch of their own or a part of another one runs.
#pragma once
#include "vidkv_common.h"

namespace vidkv {

// STREAM: a load that leaves nothing behind in the caches.
template <bool STREAM>
__device__ __forceinline__ u32x4 key_load(const u32x4* p) { return STREAM ? __builtin_nontemporal_load(p) : *p; }

// ---------------------------------------------------------------------------
// Pass 1: partial per-channel min / max over RANGE_CHUNK tokens of one head.
// 256 threads: thread (row = tid/16, col = tid%16)
// streams 16-byte pieces (8 channels) of rows row, row+16, ...; fp16 min/max
// are exact, so no precision is involved.
// ws layout: fp16 [nheads][chunks][2][128]  (min then max).
// ---------------------------------------------------------------------------
// The groups of a head dealt out evenly, per or per + 1 each (RANGE_CHUNK tokens at most), since a chunk takes much the same
// time whether it is full or not (80 heads x 8352 tokens with a last chunk of 160: 101.5 us a call, 100.0 so; 224 x 2080 71.5
// and 69.8).
struct Chunks { int n, per, extra; };
inline Chunks chunks_of(const Geom& g) { return Chunks{g.range_chunks, g.ng / g.range_chunks, g.ng % g.range_chunks}; }

struct RangeLds {
  h2 mn[16][16][4], mx[16][16][4];
};

// on = false: nothing is read or written, only the barrier is kept
template <bool STREAM>
__device__ __forceinline__ void range_part(const u32x4* __restrict__ K, int T, const Chunks& chunks,
                                           _Float16* __restrict__ ws, int chunk, long long hd, int tid,
                                           bool on, RangeLds& lds) {
  const int col = tid & 15, row = tid >> 4;
  const int t0 = G * (chunk * chunks.per + min(chunk, chunks.extra));
  const int t1 = on ? t0 + G * (chunks.per + (chunk < chunks.extra ? 1 : 0)) : 0;
  const u32x4* base = K + (hd * T) * 16 + col;   // 16 u32x4 per token row

  const _Float16 big = (_Float16)65504.0f;
  h2 mn[4], mx[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) { mn[i] = h2{big, big}; mx[i] = h2{-big, -big}; }

  int t = t0 + row;
  // 4 independent 16-byte loads in flight per thread
  for (; t + 48 < t1; t += 64) {
    U4H a, b, c, d;
    a.u = key_load<STREAM>(base + (long long)t * 16);
    b.u = key_load<STREAM>(base + (long long)(t + 16) * 16);
    c.u = key_load<STREAM>(base + (long long)(t + 32) * 16);
    d.u = key_load<STREAM>(base + (long long)(t + 48) * 16);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      mn[i] = __builtin_elementwise_min(__builtin_elementwise_min(mn[i], a.h[i]),
                                        __builtin_elementwise_min(b.h[i], c.h[i]));
      mn[i] = __builtin_elementwise_min(mn[i], d.h[i]);
      mx[i] = __builtin_elementwise_max(__builtin_elementwise_max(mx[i], a.h[i]),
                                        __builtin_elementwise_max(b.h[i], c.h[i]));
      mx[i] = __builtin_elementwise_max(mx[i], d.h[i]);
    }
  }
  for (; t < t1; t += 16) {
    U4H a;
    a.u = key_load<STREAM>(base + (long long)t * 16);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      mn[i] = __builtin_elementwise_min(mn[i], a.h[i]);
      mx[i] = __builtin_elementwise_max(mx[i], a.h[i]);
    }
  }

  h2 (&smn)[16][16][4] = lds.mn;
  h2 (&smx)[16][16][4] = lds.mx;
#pragma unroll
  for (int i = 0; i < 4; ++i) { smn[row][col][i] = mn[i]; smx[row][col][i] = mx[i]; }
  __syncthreads();
  if (on && tid < 128) {
    const int c8 = tid >> 3, e = tid & 7;
    _Float16 lo = big, hi = -big;
    for (int r = 0; r < 16; ++r) {
      const _Float16 a = smn[r][c8][e >> 1][e & 1];
      const _Float16 b = smx[r][c8][e >> 1][e & 1];
      lo = a < lo ? a : lo;
      hi = b > hi ? b : hi;
    }
    _Float16* o = ws + ((hd * chunks.n + chunk) * 2) * D;
    o[tid] = lo;
    o[D + tid] = hi;
  }
}

// The same by 1024 threads, 8 pieces in flight each: a chunk in one go, two workgroups on a compute unit.
struct ChunkRangeLds {
  h2 mn[16][16][4], mx[16][16][4];
};

template <bool STREAM>
__device__ __forceinline__ void range_chunk(const u32x4* __restrict__ K, int T, const Chunks& chunks, _Float16* __restrict__ ws,
                                            int chunk, long long hd, ChunkRangeLds& lds) {
  const int tid = threadIdx.x, col = tid & 15, row = tid >> 4;
  const int t0 = G * (chunk * chunks.per + min(chunk, chunks.extra)), t1 = t0 + G * (chunks.per + (chunk < chunks.extra ? 1 : 0));
  const u32x4* base = K + (hd * T) * 16 + col;
  const _Float16 big = (_Float16)65504.0f;
  U4H x[RANGE_CHUNK / 64];
#pragma unroll
  for (int k = 0; k < RANGE_CHUNK / 64; ++k) {       // (a row past the end repeats the first one)
    const u32x4* at = base + (long long)(t0 + row + 64 * k < t1 ? t0 + row + 64 * k : t0) * 16;
    x[k].u = key_load<STREAM>(at);
  }
  h2 mn[4], mx[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) { mn[i] = h2{big, big}; mx[i] = h2{-big, -big}; }
#pragma unroll
  for (int k = 0; k < RANGE_CHUNK / 64; ++k)
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      mn[i] = __builtin_elementwise_min(mn[i], x[k].h[i]);
      mx[i] = __builtin_elementwise_max(mx[i], x[k].h[i]);
    }
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int d = 16; d <= 32; d <<= 1) {
      mn[i] = __builtin_elementwise_min(mn[i], __builtin_bit_cast(h2, __shfl_xor(__builtin_bit_cast(int, mn[i]), d, 64)));
      mx[i] = __builtin_elementwise_max(mx[i], __builtin_bit_cast(h2, __shfl_xor(__builtin_bit_cast(int, mx[i]), d, 64)));
    }
  if ((tid & 63) < 16) {
#pragma unroll
    for (int i = 0; i < 4; ++i) { lds.mn[tid >> 6][col][i] = mn[i]; lds.mx[tid >> 6][col][i] = mx[i]; }
  }
  __syncthreads();
  if (tid < 128) {                                   // two channels' minima, or maxima
    const int c2 = tid & 63;
    h2 v = tid < 64 ? h2{big, big} : h2{-big, -big};
#pragma unroll
    for (int w = 0; w < 16; ++w) {
      const h2 y = (tid < 64 ? lds.mn : lds.mx)[w][c2 >> 2][c2 & 3];
      v = tid < 64 ? __builtin_elementwise_min(v, y) : __builtin_elementwise_max(v, y);
    }
    *reinterpret_cast<h2*>(ws + ((hd * chunks.n + chunk) * 2) * D + 2 * tid) = v;
  }
}

// ---------------------------------------------------------------------------
// Channel selection: R_c = float(max) - float(min); the n_a largest (ties to
// the lower channel) are anomalous.  perm = anomalous ascending, then normal
// ascending.  NT threads: NT / 16 slices of the chunk list, 8 channels per thread.
// ---------------------------------------------------------------------------
template <int NT>
struct ChanSelLds {
  h2 mn[NT / 64][16][4], mx[NT / 64][16][4];
  float R[D];
  int cnt0;
};

template <int NT>
__device__ __forceinline__ void select_channels(const _Float16* __restrict__ ws, int chunks, int n_a,
                                                uint8_t* __restrict__ perm, long long hd, ChanSelLds<NT>& lds) {
  constexpr int SL = NT / 16;                        // slices
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  // gather: thread (slice = tid / 16, col = tid % 16) folds 8 channels of the
  // chunks slice, slice + SL, ... with 16-byte loads, 8 chunks in flight
  const int col = tid & 15, slice = tid >> 4;
  const u32x4* p4 = reinterpret_cast<const u32x4*>(ws + hd * chunks * 2 * D) + col;
  const _Float16 big = (_Float16)65504.0f;
  h2 mn[4], mx[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) { mn[i] = h2{big, big}; mx[i] = h2{-big, -big}; }
  for (int k0 = slice; k0 < chunks; k0 += 8 * SL) {
    U4H a[8], b[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const int k = k0 + SL * u;
      const int kk = k < chunks ? k : k0;             // a repeated chunk changes nothing
      a[u].u = p4[(kk * 2) * 16];
      b[u].u = p4[(kk * 2 + 1) * 16];
    }
#pragma unroll
    for (int u = 0; u < 8; ++u)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        mn[i] = __builtin_elementwise_min(mn[i], a[u].h[i]);
        mx[i] = __builtin_elementwise_max(mx[i], b[u].h[i]);
      }
  }
  // the 4 slices of a wave (lanes 16 apart), then the waves through LDS
#pragma unroll
  for (int i = 0; i < 4; ++i) {
#pragma unroll
    for (int d = 16; d <= 32; d <<= 1) {
      mn[i] = __builtin_elementwise_min(mn[i], __builtin_bit_cast(h2, __shfl_xor(__builtin_bit_cast(int, mn[i]), d, 64)));
      mx[i] = __builtin_elementwise_max(mx[i], __builtin_bit_cast(h2, __shfl_xor(__builtin_bit_cast(int, mx[i]), d, 64)));
    }
  }
  auto& smn = lds.mn;
  auto& smx = lds.mx;
  float (&R)[D] = lds.R;
  int& cnt0 = lds.cnt0;
  if (lane < 16) {
#pragma unroll
    for (int i = 0; i < 4; ++i) { smn[wave][col][i] = mn[i]; smx[wave][col][i] = mx[i]; }
  }
  __syncthreads();
  // from here on threads 0..127 (waves 0 and 1) own one channel each; the other
  // waves only keep the barriers company
  const int c = tid & (D - 1);
  const bool own = tid < D;
  float r = 0.0f;
  if (own) {
    const int c8 = c >> 3, e = c & 7;
    _Float16 lo = big, hi = -big;
#pragma unroll
    for (int s = 0; s < NT / 64; ++s) {
      const _Float16 a = smn[s][c8][e >> 1][e & 1];
      const _Float16 b = smx[s][c8][e >> 1][e & 1];
      lo = a < lo ? a : lo;
      hi = b > hi ? b : hi;
    }
    r = (float)hi - (float)lo;
    R[c] = r;
  }
  __syncthreads();
  int an = 0, below = 0;
  if (own) {
    int rank = 0;
#pragma unroll 16
    for (int j = 0; j < D; ++j) {
      const float rj = R[j];
      rank += (rj > r || (rj == r && j < c)) ? 1 : 0;
    }
    an = rank < n_a ? 1 : 0;
  }
  // anomalous channels below mine: inside my wave by ballot, wave 0's total through LDS
  const unsigned long long bal = __ballot(an);
  below = __popcll(bal & ((1ull << lane) - 1ull));
  if (tid == 0) cnt0 = __popcll(bal);
  __syncthreads();
  if (own) {
    if (wave == 1) below += cnt0;
    const int pos = an ? below : n_a + (c - below);
    perm[hd * D + pos] = (uint8_t)c;
  }
}

// The same by 256 threads where a head has few chunks: into LDS, for a workgroup that goes on with it, and to perm where
// that is not null.  The caller's barrier lies behind it.
struct FewChanLds {
  h2 mn[16][16][4], mx[16][16][4];
  float R[D];
  int rank[2][D];
  int cnt0;
  uint8_t perm[D];
};

__device__ __forceinline__ void few_channels(const _Float16* __restrict__ ws, int chunks, int n_a, uint8_t* perm,
                                             long long hd, FewChanLds& lds) {
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, col = tid & 15, slice = tid >> 4;
  const u32x4* p4 = reinterpret_cast<const u32x4*>(ws + hd * chunks * 2 * D) + col;
  const _Float16 big = (_Float16)65504.0f;
  h2 mn[4], mx[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) { mn[i] = h2{big, big}; mx[i] = h2{-big, -big}; }
  for (int k = slice; k < chunks; k += 16) {         // (once, but for a device of many compute units)
    U4H a, b;
    a.u = p4[(k * 2) * 16];
    b.u = p4[(k * 2 + 1) * 16];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      mn[i] = __builtin_elementwise_min(mn[i], a.h[i]);
      mx[i] = __builtin_elementwise_max(mx[i], b.h[i]);
    }
  }
#pragma unroll
  for (int i = 0; i < 4; ++i) { lds.mn[slice][col][i] = mn[i]; lds.mx[slice][col][i] = mx[i]; }
  __syncthreads();
  const int c = tid & (D - 1), half = tid >> 7;
  if (half == 0) {
    const int c8 = c >> 3, e = c & 7;
    _Float16 lo = big, hi = -big;
#pragma unroll
    for (int s = 0; s < 16; ++s) {
      const _Float16 a = lds.mn[s][c8][e >> 1][e & 1];
      const _Float16 b = lds.mx[s][c8][e >> 1][e & 1];
      lo = a < lo ? a : lo;
      hi = b > hi ? b : hi;
    }
    lds.R[c] = (float)hi - (float)lo;
  }
  __syncthreads();
  const float r = lds.R[c];
  int rank = 0;
#pragma unroll
  for (int j = 0; j < D / 2; j += 4) {
    const float4 rj = *reinterpret_cast<const float4*>(&lds.R[64 * half + j]);
    const float x[4] = {rj.x, rj.y, rj.z, rj.w};
#pragma unroll
    for (int e = 0; e < 4; ++e) rank += (x[e] > r || (x[e] == r && 64 * half + j + e < c)) ? 1 : 0;
  }
  lds.rank[half][c] = rank;
  __syncthreads();
  int an = 0;
  if (half == 0) an = lds.rank[0][c] + lds.rank[1][c] < n_a ? 1 : 0;
  const unsigned long long bal = __ballot(an);
  int below = __popcll(bal & ((1ull << lane) - 1ull));
  if (tid == 0) lds.cnt0 = __popcll(bal);
  __syncthreads();
  if (half == 0) {
    if (wave == 1) below += lds.cnt0;
    const int pos = an ? below : n_a + (c - below);
    lds.perm[pos] = (uint8_t)c;
    if (perm) perm[hd * D + pos] = (uint8_t)c;
  }
}

}  // namespace vidkv
