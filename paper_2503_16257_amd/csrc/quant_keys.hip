// Key quantizer kernels (Alg. 3, MixQuant): per-channel range over all tokens,
// top-n_a channel selection, and per 32-token group the 2-bit uniform code
// (Eq. 4) of the selected channels and the sign bits of a 32-point real DFT
// (Eq. 5) of the others.
#include <algorithm>
#include <type_traits>

#include "select_keys.h"
#include "select_values.h"

namespace vidkv {

// Pass 1 as a launch of its own.  grid (range_chunks, nheads); block 1024, WHOLE (a chunk in one go), or 256.
template <bool WHOLE, bool STREAM>
__global__ __launch_bounds__(WHOLE ? 1024 : 256) void k_range_kernel(const u32x4* __restrict__ K, int T,
                                                                     Chunks chunks, _Float16* __restrict__ ws) {
  __shared__ std::conditional_t<WHOLE, ChunkRangeLds, RangeLds> lds;
  if constexpr (WHOLE) range_chunk<STREAM>(K, T, chunks, ws, blockIdx.x, blockIdx.y, lds);
  else range_part<STREAM>(K, T, chunks, ws, blockIdx.x, blockIdx.y, threadIdx.x, true, lds);
}

// Pass 1 with the protected-token selection of the same call in the first nsel workgroups: a chain of
// dependent work that needs no bandwidth, beside a pass that needs nothing else.  few: a workgroup for the tokens of each
// group (or each sequence's list), which leaves RANK and IDX to the value coding; otherwise one a sequence.  Workgroups of
// 1024 threads, a chunk each, asked for in one go; four: four chunks each, a quarter of the requests at a time.
template <bool STREAM>
__global__ __launch_bounds__(1024, 8) void k_range_select_kernel(const u32x4* __restrict__ K, int T, Chunks chunks, int total,
                                                                 int nsel, int few, int four,
                                                                 _Float16* __restrict__ ws, OneSelArgs sel) {
  __shared__ union { ChunkRangeLds range; RangeLds range4[4]; FewSelLds few; OneSelLds one; } lds;
  const int id = blockIdx.x;
  if (id < nsel) {
    __builtin_amdgcn_s_setprio(3);                   // (what the rest of the workgroups do waits for memory anyway)
    if (!few) select_one(sel, id, lds.one);
    else if (sel.scores) few_select(sel, id / sel.ng, id % sel.ng, lds.few);
    else few_list(sel, id, lds.few);
    return;
  }
  const int w = id - nsel;
  if (four) {
    const int sub = threadIdx.x >> 8, c = 4 * w + sub;
    const bool on = c < total;
    range_part<STREAM>(K, T, chunks, ws, on ? c % chunks.n : 0, on ? c / chunks.n : 0, threadIdx.x & 255, on, lds.range4[sub]);
  } else {
    range_chunk<STREAM>(K, T, chunks, ws, w % chunks.n, w / chunks.n, lds.range);
  }
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

// The range pass by 1024 threads a chunk (whole) or 256: a chunk in one go is one wait for memory instead of eight, but a
// short sequence fills little of it and the workgroup costs what it always does.  From half a chunk on, where the
// launch does not fill the device from a quarter on.  Nothing protected, 256 / 1024 threads, us: 16 heads x 128 tokens
// 11.2 / 11.1, 16 x 256 13.6 / 11.4, 16 x 512 18.4 / 12.1, 64 x 1568 24.9 / 22.4, 64 x 6272 66.5 / 65.1; 896 heads x 32 tokens
// 14.3 / 17.6, x 128 22.2 / 24.7, x 256 39.9 / 40.7, x 512 68.0 / 66.5, x 1024 118.3 / 116.7; 8192 x 32 100 / 142.
static bool whole_chunks(const Geom& g) {
  return g.T >= RANGE_CHUNK / (g.nheads * g.range_chunks <= device_cu_count() ? 4 : 2);
}

// Streaming loads in the range pass, in each of its forms, where K and as many bytes of V are more than the last-level cache
// (256 MB): plain ones then push out V, which the value coding is about to read, below it they leave K for the key coding.
// Whole calls, plain / streaming, us, on the same buffers again and again, on rotating ones, behind a kernel that wrote K,
// then V, and one that wrote V, then K:
//   16 x 4 heads x 1568 tokens, 26 MB    27.3 / 27.4   28.5 / 29.0   29.2 / 30.0   29.3 / 29.8
//   28 x 4 x 2336, 67 MB                 48.7 / 50.0   49.2 / 50.0   48.0 / 50.4   47.6 / 49.1
//   64 x 4 x 1568, 103 MB                64.8 / 65.7   64.8 / 66.6   66.7 / 68.2   64.2 / 67.6
//   28 x 4 x 4704, 135 MB                82.9 / 86.2   84.4 / 84.9   93.5 / 86.3   83.4 / 85.7
//   28 x 4 x 6272, 180 MB               104.9 / 107.7 110.1 / 107.5 124.4 / 108.9 109.1 / 110.9
//   4 x 196000 (token selection beside), 201 MB   124.9 / 127.4   125.3 / 128.3   147.4 / 138.1   136.6 / 136.0
//   28 x 4 x 8192, 235 MB               136.2 / 135.9 140.3 / 138.2 160.7 / 139.6 151.6 / 141.9
//   64 x 4 x 25088, 1644 MB               889 / 886     875 / 877     906 / 889     908 / 887
// So what is read behind a kernel that wrote V last decides; on the same or rotating buffers a call between 128 and 256 MiB loses
// up to 3 % by it.  Plain loads for the last 32 to 128 MiB alone lie between the two in each column.
static bool stream_keys(const Geom& g) { return (size_t)g.nheads * g.T * D * 2 > ((size_t)128 << 20); }

// Counting the tokens with larger scores, quadratic in the sequence, against one workgroup's four digits: up to 8192 tokens on
// each compute unit's share (the selection by itself, 256 groups of one sequence, whole calls: 20.2 us with the digits, 17.0; of
// two 22.4 and 22.9; 2 x 8 heads x 8128 tokens, 16129 a unit, 34.3 and 36.0); beside a range pass, which waits for its workgroups, while
// they and the chunks are no more than three a compute unit (digits and counting, us: 8 x 4 heads x 1568 tokens, 520, 21.8 and
// 19.9; 2 x 8 x 4704, 454, 25.4 and 23.2; 56 x 4 x 256, 672, 22.4 and 18.9; 32 x 4 x 512 in 2 layers, 768, 30.2 and 29.3; 8 x 4 x 288 in
// 16, 656, 33.6 and 34.2; 64 x 4 x 288, 832, 24.0 and 25.8; 8 x 4 x 1568 in 8, 1416, 64.3 and 68.7; 64 x 8 x 544, 2112, 50.2 and 57.9.
// Where 256 threads take a chunk, the line is at one and a half, four chunks counted as one: 32 x 4 x 64 tokens in 8 layers, 320,
// 26.8 and 24.7; 64 x 4 x 160, 384, 21.9 and 19.4; 32 x 4 x 160 in 8, 416, 41.8 and 43.7; 64 x 4 x 64 in 8, 640, 41.3 and 42.0.)
// A list's selection is quick, but ranks and IDX then cost the value coding a little of each group: the same line.
bool few_selection(const Geom& g, bool scores, bool alone) {
  if (g.ng > FEW_MAX_GROUPS) return false;
  const long long cus = device_cu_count(), nsel = scores ? (long long)g.B * g.ng : g.B, chunks = g.nheads * g.range_chunks;
  if (scores && nsel * g.T > 8192 * cus) return false;
  if (alone) return true;
  return whole_chunks(g) ? nsel + chunks <= 3 * cus : 2 * nsel + (chunks + 1) / 2 <= 3 * cus;
}

// The range pass (Range metric) and the protected-token selection of short sequences (or none) in one launch.
// few: few_selection(), and the value coding finds RANK and IDX.
void launch_k_range_select(const Geom& g, const void* K, void* ws, const float* scores, const int32_t* idx,
                           uint8_t* packed_V, bool few, hipStream_t st) {
  const int nsel = g.n_s == 0 ? 0 : few && scores ? g.B * g.ng : g.B;
  const long long total = g.nheads * g.range_chunks, cus = device_cu_count();
  // Beside a workgroup that goes through a sequence's digits, four chunks a workgroup also where the chunks are not nearly
  // full (64 x 4 heads x 544 tokens in 8 layers 169 us so, 179 with a chunk each; 16 x 4 x 3136, 0.88 full, 43.4 and 40.9), and where
  // the selection is the longer part and so keeps a compute unit to itself: K and V just written, 4 x 4 heads x 6272 tokens, 208
  // chunks, 30.2 and 31.5, 4 x 8 x 6272, 416, 38.8 and 40.7, 6 x 8 x 6272, 624, 52.8 and 51.5; 2 x 8 x 8192, 256, 33.4 and 35.8, 8 x 4 x
  // 8192, 512, 49.6 and 46.4; 4 x 8 x 12544, 800, 72.2 and 73.7, 8 heads of 25088, 392, 51.0 and 54.0, 16 of 32768, 1024, 99.1 and 94.2.
  const bool digits = nsel > 0 && !few;
  const bool four = !whole_chunks(g) || (digits && 8LL * g.T < 7LL * RANGE_CHUNK * g.range_chunks) ||
                    (digits && g.T > 16 * FEW_MAX_GROUPS && 4 * total <= 7 * cus) ||
                    (digits && g.T > 32 * FEW_MAX_GROUPS && (total + 3) / 4 + nsel <= cus);
  const long long wgs = four ? (total + 3) / 4 : total;
  // T <= ONE_MAX_T: at most 65535 * 64 chunks
  hipLaunchKernelGGL(stream_keys(g) ? k_range_select_kernel<true> : k_range_select_kernel<false>, dim3((unsigned)(nsel + wgs)), dim3(1024), 0, st,
                     reinterpret_cast<const u32x4*>(K), g.T, chunks_of(g), (int)total, nsel, few ? 1 : 0, four ? 1 : 0,
                     reinterpret_cast<_Float16*>(ws), one_sel_args(g, scores, idx, packed_V));
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
  if (stages & 1u) {
    const bool whole = whole_chunks(g), stream = stream_keys(g);
    auto* kernel = whole ? (stream ? k_range_kernel<true, true> : k_range_kernel<true, false>)
                         : (stream ? k_range_kernel<false, true> : k_range_kernel<false, false>);
    hipLaunchKernelGGL(kernel, gr1, dim3(whole ? 1024 : 256), 0, st, k4, g.T, chunks_of(g), w);
  }
  if (stages & 2u)
    hipLaunchKernelGGL(k_select_kernel, dim3((unsigned)g.nheads), dim3(1024), 0, st, w,
                       g.range_chunks, g.n_a, packed + g.k_perm);
  if (stages & 4u)
    launch_k_encode(g, EncodeSpan{g.T, g.ng, 0, g.nheads, 0}, K, packed, g.use_fft, st);
  return hipGetLastError();
}

}  // namespace vidkv
