// Decode attention over the packed cache (Eq. 3; Alg. 1, Decoding):
// split-T partial softmax-attention with the dequantization fused in, then a
// log-sum-exp merge.  The dequantized K', V' never exist in memory.
//
// Normal key channels are scored in the frequency domain: by linearity
//   sum_c q_c IDFT(Xhat_c)[t] = IDFT(sum_c q_c Xhat_c)[t],
// so per 32-token group the +-s coefficients are contracted over channels first
// (Y[h][slot]) and a single 32-point inverse real DFT per query head follows.
//
// This file holds the merge kernel and the launcher; the fp16 residual tokens' part is in
// decode_attn.h, the MFMA kernel that reads the packed tokens in decode_attn_mfma.h.
#include "decode_attn.h"

#include <algorithm>
#include <atomic>

namespace vidkv {

// The residual tokens as a launch of their own (the MFMA kernel takes them along when its grid
// has room for them).
__global__ __launch_bounds__(256, 3) void attn_tail_kernel(AttnArgs a) {
  __shared__ TailLds t;
  attn_tail_part(a, blockIdx.x, blockIdx.y, blockIdx.z, t);
}

// Merge of the split partials: out = sum_i o_i 2^{m_i - M} / sum_i l_i 2^{m_i - M}.
// grid (Hq, B), block 256 = 32 channel quads x 8 slices of the list of parts.  What takes time is
// latency - the launch, the round trips to memory, the reduction - so everything is asked for at once: the
// arguments, then up to 8 U parts, 16 bytes of a part per thread, and their (m, l), before any is waited for.
// (As the compiler orders it by itself - arguments in two steps, (m, l) waited for in front of the sums, the sums behind
// the maximum, three to ten round trips - the kernel took 3.4 us at 28 rows x 26 parts and 4.2 at 28 x 129 x 7; so 2.8 and
// 3.8: a step of 28 layers x 6272 tokens 314 -> 299 us, one layer of 196000 28.3 -> 27.4, 28 x 8 x 12544 485 -> 476.)
template <int U>
__global__ __launch_bounds__(256) void attn_merge_kernel(const float* __restrict__ part_o,
                                                         const float2* __restrict__ part_ml,
                                                         int nparts, int BHq,
                                                         _Float16* __restrict__ out) {
  asm volatile("" :: "s"(part_o), "s"(part_ml), "s"(nparts), "s"(BHq), "s"(out));
  const int row = blockIdx.y * gridDim.x + blockIdx.x;             // (sequence, query head)
  const int c4 = threadIdx.x & 31, sl = threadIdx.x >> 5;
  __shared__ f4 so[8][32];
  __shared__ float sl_[8], sM[8];
  const f4* po = reinterpret_cast<const f4*>(part_o) + (size_t)row * (D / 4) + c4;
  const float2* pm = part_ml + row;
  f4 o = f4{0.f, 0.f, 0.f, 0.f};
  float l = 0.0f, M = -INFINITY;
  // slice sl takes parts sl, sl + 8, ...; its sums are relative to its own running maximum
  for (int i0 = sl; i0 < nparts; i0 += 8 * U) {
    f4 oi[U];
    float2 ml[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int i = i0 + 8 * u, ii = i < nparts ? i : i0;          // (past the end: a part again, not counted)
      ml[u] = pm[(size_t)ii * BHq];
      oi[u] = po[(size_t)ii * BHq * (D / 4)];
    }
    // (left to itself the compiler waits for (m, l) first, and for the sums only behind the maximum)
#pragma unroll
    for (int u = 0; u < U; ++u) asm volatile("" : "+v"(oi[u]), "+v"(ml[u].x), "+v"(ml[u].y));
    float Mn = M;
#pragma unroll
    for (int u = 0; u < U; ++u) {
      if (i0 + 8 * u >= nparts) ml[u].x = -INFINITY;
      Mn = fmaxf(Mn, ml[u].x);
    }
    const float w0 = M == -INFINITY ? 0.0f : __builtin_amdgcn_exp2f(M - Mn);
    o *= w0;
    l *= w0;
    M = Mn;
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const float w = ml[u].x == -INFINITY ? 0.0f : __builtin_amdgcn_exp2f(ml[u].x - M);
      const bool any = w != 0.0f;                                  // an empty part's sums are never looked at
#pragma unroll
      for (int e = 0; e < 4; ++e) o[e] += any ? w * oi[u][e] : 0.0f;
      l += any ? w * ml[u].y : 0.0f;
    }
  }
  so[sl][c4] = o;
  if (c4 == 0) { sl_[sl] = l; sM[sl] = M; }
  __syncthreads();
  if (threadIdx.x < D) {
    const int c = threadIdx.x;
    float Mx = sM[0];
#pragma unroll
    for (int i = 1; i < 8; ++i) Mx = fmaxf(Mx, sM[i]);
    float acc = 0.0f, L = 0.0f;
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const float w = sM[i] == -INFINITY ? 0.0f : __builtin_amdgcn_exp2f(sM[i] - Mx);
      acc += w * so[i][c >> 2][c & 3];
      L += w * sl_[i];
    }
    out[(size_t)row * D + c] = (_Float16)(L > 0.0f ? acc / L : 0.0f);
  }
}

// Compute units of the current device, asked once per device. A process with no usable
// device (a size query on a build host) gets the MI355X figure, 256.
int device_cu_count() {
  constexpr int MAXDEV = 64;
  static std::atomic<int> cached[MAXDEV];
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= MAXDEV) {
    (void)hipGetLastError();
    return 256;
  }
  int n = cached[dev].load(std::memory_order_relaxed);
  if (n > 0) return n;
  if (hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n <= 0) {
    (void)hipGetLastError();
    n = 256;
  }
  cached[dev].store(n, std::memory_order_relaxed);
  return n;
}

// Split-T workgroups per (sequence, KV head) that every accepted workspace has room for: one round
// of workgroups, two pairs per wave.
int attn_least_splits(const Geom& g) {
  if (g.ng == 0) return 0;
  const long long bh = (long long)g.B * g.H, npairs = (g.ng + 1) / 2, cus = device_cu_count();
  return (int)std::max(1LL, std::min((2 * cus + bh - 1) / bh, (npairs + 7) / 8));
}

// The most that attn_splits() can choose: what the workspace is sized for.  Grows with the number of
// groups.  One pair per wave and two rounds of workgroups, but not so many that the partials outgrow
// the array of the entry point without a workspace - unless the least number already does.
int attn_max_splits(const Geom& g) {
  if (g.ng == 0) return 0;
  const long long bh = (long long)g.B * g.H, npairs = (g.ng + 1) / 2, cus = device_cu_count();
  const long long fit = ((long long)VIDKV_NOALLOC_SCRATCH_BYTES - 512) / ((long long)g.B * g.Hq * (D + 2) * 4) - ATTN_TAIL_SPLITS;
  return (int)std::max((long long)attn_least_splits(g), std::min({(npairs + 3) / 4, 4 * cus / bh, fit}));
}

// The costs below are in 0.1 us: of a round of workgroups, two resident per compute unit, that take s
// pairs of groups one after another in each of 4 waves; 6 us to get going and finish, 2.2 us per pair where a
// compute unit has one workgroup, 3.5 where it has two.  Fitted at n_a = 64 to a kernel that took that long (the
// split chosen cost 0.6 % more than the fastest tried on average, 16 % at most) and kept: later ones get
// going earlier and spend fewer instructions on a pair, and choose as well (n_a = 64, 16 with fp16 rows, 96, and 64 with
// 2-bit rows, 1 to 64 sequences x 4 heads of 192 to 12544 tokens, 420 shapes: 1.8 % over the fastest tried; with residual
// tokens: attn_plan()).
static long long main_cost(int s, int w, int cus) {
  // a 64-bit product: thousands of rounds of thousands of pairs
  return (long long)((w + 2 * cus - 1) / (2 * cus)) * (60 + (long long)s * (w <= cus ? 22 : 35));
}

// Split-T workgroups per (sequence, KV head), nmax at most, in a launch without residual tokens: tried are all
// s up to 64, then the even split over one round.  (A fixed aim of two workgroups per unit
// and at least 2 pairs per wave took 2.2 us more where there are few pairs, a second, nearly empty
// round where 512 / (B H) is no whole number, and more workgroups than needed for the same s.)
static int attn_splits(int bh, int npairs, int nmax, int cus, long long* cost) {
  // 32-bit arithmetic: the candidates' divisions are on every decode call's way
  int best_n = 1;
  long long best_t = -1;
  auto consider = [&](int n) {
    if (n < 1 || n > nmax) return;
    const long long t = main_cost(((npairs + n - 1) / n + 3) / 4, n * bh, cus);
    if (best_t < 0 || t < best_t) { best_t = t; best_n = n; }
  };
  consider(std::min(std::max(1, 2 * cus / bh), nmax));
  for (int s = std::min(64, (npairs + 3) / 4); s >= 1; --s) {
    const int n = (npairs + 4 * s - 1) / (4 * s);
    if (n > nmax) break;
    consider(n);
  }
  *cost = best_t;
  return best_n;
}

struct AttnPlan {
  int nsplit, ntail;   // workgroups per (sequence, KV head): packed tokens, residual tokens
  bool along;          // the latter in the same launch
};

// `iters` blocks of 32 residual tokens per head, a wave of a residual workgroup one or more of them, `turns` one
// after another.  In the same launch, where all workgroups fit one round, their time disappears behind the packed
// tokens': 3.5 us and 2.2 us a turn, 3.2 where a compute unit has two workgroups.  A launch of its own costs 7.0 us
// and 2.8 us a turn and round of three workgroups a compute unit.  Fitted to 780 shapes (1 to 64 sequences x 1 to 8
// heads of 192 to 12544 tokens, 32 to 1024 residual ones, four variants), main_cost() as it is: 1.3 % over the fastest split tried on
// average, 29 % at most (on residual workgroups 1 to 4 % faster at 1024 tokens, whose probabilities had fewer bits).  Large
// blocks, too (64 x 4 heads x 25088 tokens, 256 residual ones: the launch takes 6.9 us; on a stream of its own beside
// the packed tokens' the call took 147 us, behind them 140).
static AttnPlan attn_plan(const Geom& g, int nmax, int iters) {
  const int bh = (int)std::min((long long)g.B * g.H, 1LL << 20), cus = device_cu_count(), npairs = (g.ng + 1) / 2;
  const int ntail = std::min((iters + 3) / 4, ATTN_TAIL_SPLITS);
  AttnPlan best{0, ntail, false};
  long long best_t = -1, own = 0;
  if (iters > 0) {
    const int turns0 = (iters + 4 * ntail - 1) / (4 * ntail);
    own = 70 + 28LL * turns0 * (((long long)bh * ntail + 3 * cus - 1) / (3 * cus));
    // from the most workgroups down to the fewest; of the splits that fit beside them in
    // one round, or in one workgroup per compute unit, the finest
    for (int nt = ntail, turns = turns0;;) {
      for (int room = 2; room >= 1; --room) {
        const int most = std::min(nmax, room * cus / bh - nt);
        if (most < 1) continue;
        const int s = ((npairs + most - 1) / most + 3) / 4;
        const int n = room == 2 ? most : (npairs + 4 * s - 1) / (4 * s), w = bh * (n + nt);
        const long long t = std::max(main_cost(s, w, cus), 35 + (long long)turns * (w <= cus ? 22 : 32));
        // of equal costs the finer split: fewer of its waves take the last of the s pairs
        if (best_t < 0 || t < best_t || (t == best_t && n > best.nsplit)) { best_t = t; best = {n, nt, true}; }
      }
      if (nt == 1) break;
      turns = (iters + 4 * (nt - 1) - 1) / (4 * (nt - 1));   // the next smaller number that changes the blocks per wave
      nt = (iters + 4 * turns - 1) / (4 * turns);
    }
  }
  if (best_t < 0 || best_t > 82 + own) {               // 82: the least that main_cost() can be
    long long t;
    const int n = attn_splits(bh, npairs, nmax, cus, &t);
    if (best_t < 0 || t + own < best_t) best = {n, ntail, false};
  }
  return best;
}

// ws_bytes: room for attn_least_splits() + ATTN_TAIL_SPLITS parts at least.
hipError_t launch_decode_attention(const Geom& g, int layer, float scale, const void* q,
                                   const uint8_t* pk, const uint8_t* pv, const void* ktail,
                                   const void* vtail, int cap, const int32_t* tail_len, void* out,
                                   void* ws, size_t ws_bytes, unsigned stages, hipStream_t st) {
  AttnArgs a;
  a.q = reinterpret_cast<const _Float16*>(q);
  a.kperm = pk + g.k_perm;
  a.krec = pk + g.k_rec;
  a.vrec = pv + g.v_rec;
  a.vmask = reinterpret_cast<const uint32_t*>(pv + g.v_mask);
  a.vrank = reinterpret_cast<const uint32_t*>(pv + g.v_rank);
  a.vrows = reinterpret_cast<const _Float16*>(pv + g.v_rows);
  a.ktail = reinterpret_cast<const _Float16*>(ktail);
  a.vtail = reinterpret_cast<const _Float16*>(vtail);
  const bool has_tail = cap > 0 && ktail && vtail && tail_len;
  a.tail_len = has_tail ? tail_len : nullptr;
  a.layer = layer; a.B = g.B; a.H = g.H; a.Hq = g.Hq; a.rep = g.rep; a.ng = g.ng; a.ngc = g.ngc;
  a.n_a = g.n_a; a.n_s = g.n_s; a.cap = cap;
  a.sal_bits = g.sal_bits; a.npg = g.npg; a.use_fft = g.use_fft ? 1 : 0;
  a.scale2 = scale * 1.4426950408889634f;
  // stages: bit 0 split-T partial kernel(s), bit 1 merge
  // Residual tokens: in the MFMA kernel's launch, or in one of their own behind it.
  // With no token at all one empty part per head is still written.
  const long long bh = (long long)g.B * g.H, slots = 2LL * device_cu_count();
  const int tail_iters = has_tail ? (cap + 31) / 32 : 0;
  const long long fit = (long long)(ws_bytes / ((size_t)g.B * g.Hq * (D + 2) * sizeof(float))) - ATTN_TAIL_SPLITS;
  const int nmax = (int)std::min((long long)attn_max_splits(g), fit);
  int ntail = std::max(1, std::min((tail_iters + 3) / 4, ATTN_TAIL_SPLITS));
  bool along = false;
  a.nsplit = 0;
  if (g.ng > 0) {
    const AttnPlan p = attn_plan(g, nmax, tail_iters);
    a.nsplit = p.nsplit;
    ntail = p.ntail;
    along = p.along;
  }
  a.early = bh * (a.nsplit + (along ? ntail : 0)) <= slots / 2;
  a.tail_per = ntail > 0 && tail_iters > 0 ? (tail_iters + ntail - 1) / ntail : 0;
  const int nparts = a.nsplit + ntail;
  a.part_o = reinterpret_cast<float*>(ws);                        // 16-byte aligned rows
  a.part_ml = a.part_o + (size_t)nparts * g.B * g.Hq * D;
  if (stages & 1u) {
    const int npairs = (g.ng + 1) / 2;
    a.gps = a.nsplit > 0 ? (npairs + a.nsplit - 1) / a.nsplit : 0;   // pairs per split
    const dim3 gtail(ntail, g.H, g.B), gmain(a.nsplit + (along ? ntail : 0), g.H, g.B);
    if (a.nsplit > 0) launch_attn_mfma(a, gmain, st);
    if (ntail > 0 && !along) hipLaunchKernelGGL(attn_tail_kernel, gtail, dim3(256), 0, st, a);
  }
  if (stages & 2u) {
    _Float16* o16 = reinterpret_cast<_Float16*>(out);
    const dim3 gm(g.Hq, g.B);
    const int BHq = g.B * g.Hq;
    const float2* ml = reinterpret_cast<const float2*>(a.part_ml);
    if (nparts <= 16)
      hipLaunchKernelGGL(attn_merge_kernel<2>, gm, dim3(256), 0, st, a.part_o, ml, nparts, BHq, o16);
    else if (nparts <= 32)
      hipLaunchKernelGGL(attn_merge_kernel<4>, gm, dim3(256), 0, st, a.part_o, ml, nparts, BHq, o16);
    else if (nparts <= 72)
      hipLaunchKernelGGL(attn_merge_kernel<9>, gm, dim3(256), 0, st, a.part_o, ml, nparts, BHq, o16);
    else
      hipLaunchKernelGGL(attn_merge_kernel<17>, gm, dim3(256), 0, st, a.part_o, ml, nparts, BHq, o16);
  }
  return hipGetLastError();
}

}  // namespace vidkv
