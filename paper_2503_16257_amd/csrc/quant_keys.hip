// Key quantizer kernels (Alg. 3, MixQuant): per-channel range over all tokens,
// top-n_a channel selection, and per 32-token group the 2-bit uniform code
// (Eq. 4) of the selected channels and the sign bits of a 32-point real DFT
// (Eq. 5) of the others.
#include "select_keys.h"
#include "select_values.h"

namespace vidkv {

// Pass 1 as a launch of its own.  grid (range_chunks, nheads), block 256.
__global__ __launch_bounds__(256) void k_range_kernel(const u32x4* __restrict__ K, int T,
                                                      int chunks, _Float16* __restrict__ ws) {
  __shared__ RangeLds lds;
  range_part(K, T, chunks, ws, blockIdx.x, blockIdx.y, threadIdx.x, true, lds);
}

// Pass 1 with the protected-token selection of the same call in the first B workgroups: a chain of
// dependent work that needs no bandwidth, beside a pass that needs nothing else.  Workgroups of
// 1024 threads, four chunks each.
// (28 x 6272 tokens: range pass 29 us, then six selection launches of 4.7 us; both in one 31.4.)
__global__ __launch_bounds__(1024, 8) void k_range_select_kernel(const u32x4* __restrict__ K, int T,
                                                                 int chunks, int total, int B,
                                                                 _Float16* __restrict__ ws, OneSelArgs sel) {
  __shared__ union { RangeLds range[4]; OneSelLds one; } lds;
  if ((int)blockIdx.x < B) {
    select_one(sel, blockIdx.x, lds.one);
    return;
  }
  const int sub = threadIdx.x >> 8;
  const int id = (blockIdx.x - B) * 4 + sub;
  const bool on = id < total;
  range_part(K, T, chunks, ws, on ? id % chunks : 0, on ? id / chunks : 0, threadIdx.x & 255, on, lds.range[sub]);
}

// Calls with few groups: the ranges of all chunks, and a workgroup for the protected tokens of each group (or
// each sequence's list), in one launch.
__global__ __launch_bounds__(1024) void k_few_first_kernel(const u32x4* __restrict__ K, int T, int chunks, int nsel,
                                                           _Float16* __restrict__ ws, OneSelArgs sel) {
  __shared__ union { FewRangeLds range; FewSelLds sel; } lds;
  const int id = blockIdx.x;
  if (id < nsel) {
    if (sel.scores) few_select(sel, id / sel.ng, id % sel.ng, lds.sel);
    else few_list(sel, id, lds.sel);
    return;
  }
  few_range(K, T, chunks, ws, (id - nsel) % chunks, (id - nsel) / chunks, lds.range);
}

// Channel selection as a launch of its own.  grid nheads, block 1024.
__global__ __launch_bounds__(1024) void k_select_kernel(const _Float16* __restrict__ ws,
                                                        int chunks, int n_a,
                                                        uint8_t* __restrict__ perm) {
  __shared__ ChanSelLds<1024> lds;
  select_channels<1024>(ws, chunks, n_a, perm, blockIdx.x, lds);
}

// ---------------------------------------------------------------------------
// The two other channel metrics of Sec. 3.2 (1), both in float64 so that the
// ranking does not depend on the summation order beyond the last bits:
//   variance   sigma^2 = mean(x^2) - mean(x)^2 over all tokens of the channel
//   outliers   N = #{ t : |x_t| > M * mean|x| },  M = 3
// k_metric_kernel<MODE> writes per (head, chunk) partials double [2][128]:
//   MODE 0: sum x, sum x^2      MODE 1: sum |x|, 0      MODE 2: count(|x| > thr), 0
// grid (range_chunks, nheads), block 256: thread (row = tid / 16, col = tid % 16)
// takes 8 channels of rows row, row + 16, ... of its chunk.
// ---------------------------------------------------------------------------
template <int MODE>
__global__ __launch_bounds__(256) void k_metric_kernel(const u32x4* __restrict__ K, int T,
                                                       int chunks, const double* __restrict__ thr,
                                                       double* __restrict__ part) {
  const int chunk = blockIdx.x;
  const long long hd = blockIdx.y;
  const int tid = threadIdx.x, col = tid & 15, row = tid >> 4;
  const int t1 = min(T, (chunk + 1) * RANGE_CHUNK);
  const u32x4* base = K + (hd * T) * 16 + col;
  double a[8], b[8], th[8];
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    a[e] = 0.0; b[e] = 0.0;
    th[e] = MODE == 2 ? thr[hd * D + 8 * col + e] : 0.0;
  }
  // 8 rows requested at a time, added in ascending order (one at a time the pass waited for memory at
  // every row; with the fold below, one 196000-token layer: variance 229 -> 137 us a call, outliers
  // 354 -> 169; one head of 1568 tokens 27.1 -> 24.7 and 38.3 -> 33.4)
  for (int t0 = chunk * RANGE_CHUNK + row; t0 < t1; t0 += 128) {
    U4H x[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) x[u].u = __builtin_nontemporal_load(base + (long long)min(t0 + 16 * u, T - 1) * 16);
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      if (t0 + 16 * u < t1) {
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          const double v = (double)(float)x[u].e[e];
          if (MODE == 0) { a[e] += v; b[e] = fma(v, v, b[e]); }
          if (MODE == 1) a[e] += fabs(v);
          if (MODE == 2) a[e] += fabs(v) > th[e] ? 1.0 : 0.0;
        }
      }
    }
  }
  __shared__ double sa[16][D], sb[16][D];
#pragma unroll
  for (int e = 0; e < 8; ++e) { sa[row][8 * col + e] = a[e]; sb[row][8 * col + e] = b[e]; }
  __syncthreads();
  if (tid < D) {
    double x = 0.0, y = 0.0;
    for (int r = 0; r < 16; ++r) { x += sa[r][tid]; y += sb[r][tid]; }
    double* o = part + ((hd * chunks + chunk) * 2) * D;
    o[tid] = x;
    o[D + tid] = y;
  }
}

// Folds the partials of one head.  MODE 1: writes the outlier threshold M * mean|x| per channel.
// MODE 0 / 2: ranks the channels by variance / outlier count (ties to the lower channel) and writes
// PERM like k_select_kernel.  grid nheads, block 1024: thread = (slice of the chunks, channel); slice
// s folds chunks s, s + 8, ... in ascending order, then the slices are added in order.  (One thread
// per channel over all chunks was a chain of one memory round trip per chunk.)
template <int MODE>
__global__ __launch_bounds__(1024) void k_metric_select_kernel(const double* __restrict__ part,
                                                              int chunks, int T, int n_a,
                                                              double* __restrict__ thr,
                                                              uint8_t* __restrict__ perm) {
  const long long hd = blockIdx.x;
  const int c = threadIdx.x & (D - 1), sl = threadIdx.x >> 7;
  double x = 0.0, y = 0.0;
  for (int k0 = sl; k0 < chunks; k0 += 32) {
    double px[4], py[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int k = min(k0 + 8 * u, chunks - 1);
      px[u] = part[((hd * chunks + k) * 2) * D + c];
      py[u] = MODE == 0 ? part[((hd * chunks + k) * 2 + 1) * D + c] : 0.0;
    }
#pragma unroll
    for (int u = 0; u < 4; ++u)
      if (k0 + 8 * u < chunks) { x += px[u]; y += py[u]; }
  }
  __shared__ double sx[8][D], sy[8][D];
  sx[sl][c] = x;
  sy[sl][c] = y;
  __syncthreads();
  x = y = 0.0;
#pragma unroll
  for (int i = 0; i < 8; ++i) { x += sx[i][c]; y += sy[i][c]; }   // every slice's threads: the same sums
  if (MODE == 1) {
    if (sl == 0) thr[hd * D + c] = 3.0 * (x / (double)T);
    return;
  }
  const double mean = x / (double)T;
  const double r = MODE == 0 ? y / (double)T - mean * mean : x;
  __shared__ double R[D];
  __shared__ int rk[8][D];
  __shared__ int cnt0;
  if (sl == 0) R[c] = r;
  __syncthreads();
  // channels that come before mine: slice sl compares with channels 16 sl .. 16 sl + 15
  int before = 0;
#pragma unroll
  for (int j = 16 * sl; j < 16 * sl + 16; ++j) {
    const double rj = R[j];
    before += (rj > r || (rj == r && j < c)) ? 1 : 0;
  }
  rk[sl][c] = before;
  __syncthreads();
  int an = 0, below = 0;
  if (sl == 0) {
    int rank = 0;
#pragma unroll
    for (int i = 0; i < 8; ++i) rank += rk[i][c];
    an = rank < n_a ? 1 : 0;
  }
  const unsigned long long bal = __ballot(an);
  below = __popcll(bal & ((1ull << (c & 63)) - 1ull));
  if (threadIdx.x == 0) cnt0 = __popcll(bal);
  __syncthreads();
  if (sl == 0) {
    if (c >= 64) below += cnt0;
    perm[hd * D + (an ? below : n_a + (c - below))] = (uint8_t)c;
  }
}

// The per-group coding pass (Eq. 4 and Eq. 5) lives in quant_keys_mfma.hip.
void launch_k_encode(const Geom& g, const EncodeSpan& sp, const void* K, uint8_t* packed,
                     bool use_fft, hipStream_t st);

// The range pass (Range metric) and the protected-token selection of short sequences in one launch.
void launch_k_range_select(const Geom& g, const void* K, void* ws, const float* scores, const int32_t* idx,
                           uint8_t* packed_V, hipStream_t st) {
  const int total = (int)(g.nheads * g.range_chunks);            // T <= ONE_MAX_T: at most 65535 * 64
  hipLaunchKernelGGL(k_range_select_kernel, dim3(g.B + (total + 3) / 4), dim3(1024), 0, st,
                     reinterpret_cast<const u32x4*>(K), g.T, g.range_chunks, total, g.B,
                     reinterpret_cast<_Float16*>(ws), one_sel_args(g, scores, idx, packed_V));
}

void launch_k_few_first(const Geom& g, const void* K, void* ws, const float* scores, const int32_t* idx,
                        uint8_t* packed_V, hipStream_t st) {
  const int nsel = g.n_s == 0 ? 0 : scores ? g.B * g.ng : g.B;
  hipLaunchKernelGGL(k_few_first_kernel, dim3(nsel + (unsigned)(g.nheads * g.range_chunks)), dim3(1024), 0, st,
                     reinterpret_cast<const u32x4*>(K), g.T, g.range_chunks, nsel, reinterpret_cast<_Float16*>(ws),
                     one_sel_args(g, scores, idx, packed_V));
}

// ---------------------------------------------------------------------------
// stages: bit 0 range pass, bit 1 channel selection, bit 2 coding pass
hipError_t launch_quantize_keys(const Geom& g, const void* K, uint8_t* packed, void* ws,
                                unsigned stages, hipStream_t st) {
  if (g.T == 0) return hipSuccess;
  _Float16* w = reinterpret_cast<_Float16*>(ws);
  dim3 gr1(g.range_chunks, (unsigned)g.nheads);
  const u32x4* k4 = reinterpret_cast<const u32x4*>(K);
  if (g.metric != 0) {
    // variance / outlier count (the paper's ablation; Range is what it adopts): float64
    // partials [nheads][chunks][2][128], then the thresholds [nheads][128]
    double* part = reinterpret_cast<double*>(ws);
    double* thr = part + (size_t)g.nheads * g.range_chunks * 2 * D;
    dim3 gh((unsigned)g.nheads);
    if (g.metric == 1) {
      if (stages & 1u)
        hipLaunchKernelGGL(k_metric_kernel<0>, gr1, dim3(256), 0, st, k4, g.T, g.range_chunks, thr, part);
      if (stages & 2u)
        hipLaunchKernelGGL(k_metric_select_kernel<0>, gh, dim3(1024), 0, st, part, g.range_chunks, g.T,
                           g.n_a, thr, packed + g.k_perm);
    } else {
      if (stages & 1u) {
        hipLaunchKernelGGL(k_metric_kernel<1>, gr1, dim3(256), 0, st, k4, g.T, g.range_chunks, thr, part);
        hipLaunchKernelGGL(k_metric_select_kernel<1>, gh, dim3(1024), 0, st, part, g.range_chunks, g.T,
                           g.n_a, thr, packed + g.k_perm);
        hipLaunchKernelGGL(k_metric_kernel<2>, gr1, dim3(256), 0, st, k4, g.T, g.range_chunks, thr, part);
      }
      if (stages & 2u)
        hipLaunchKernelGGL(k_metric_select_kernel<2>, gh, dim3(1024), 0, st, part, g.range_chunks, g.T,
                           g.n_a, thr, packed + g.k_perm);
    }
    if (stages & 4u)
      launch_k_encode(g, EncodeSpan{g.T, g.ng, 0, g.nheads, 0}, K, packed, g.use_fft, st);
    return hipGetLastError();
  }
  if (stages & 1u)
    hipLaunchKernelGGL(k_range_kernel, gr1, dim3(256), 0, st, k4, g.T, g.range_chunks, w);
  if (stages & 2u)
    hipLaunchKernelGGL(k_select_kernel, dim3((unsigned)g.nheads), dim3(1024), 0, st, w,
                       g.range_chunks, g.n_a, packed + g.k_perm);
  if (stages & 4u)
    launch_k_encode(g, EncodeSpan{g.T, g.ng, 0, g.nheads, 0}, K, packed, g.use_fft, st);
  return hipGetLastError();
}

}  // namespace vidkv
