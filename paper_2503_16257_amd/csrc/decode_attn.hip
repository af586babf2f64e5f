// Decode attention over the packed cache (Eq. 3; Alg. 1, Decoding):
// split-T partial softmax-attention with the dequantization fused in, then a
// log-sum-exp merge.  The dequantized K', V' never exist in memory.
//
// Normal key channels are scored in the frequency domain: by linearity
//   sum_c q_c IDFT(Xhat_c)[t] = IDFT(sum_c q_c Xhat_c)[t],
// so per 32-token group the +-s coefficients are contracted over channels first
// (Y[h][slot]) and a single 32-point inverse real DFT per query head follows.
//
// This file holds the kernel for the fp16 residual tokens, the merge kernels and
// the launcher; the MFMA kernel that reads the packed tokens is in decode_attn_mfma.h.
#include "decode_attn.h"
#include <atomic>

namespace vidkv {

// The fp16 residual tokens (Alg. 1's X_Kr, X_Vr): one workgroup = one (tail split, KV head,
// sequence); split ts takes the 32-token steps ts * tail_per .. of the buffer and writes its
// partial (o, m, l) as split index nsplit + ts.  Thread roles: scores (token = tid % 32,
// head = tid / 32), output (channel = tid % 128, heads tid / 128 + 2 i).
__global__ __launch_bounds__(256) void attn_tail_kernel(AttnArgs a) {
  const int ts = blockIdx.x, kvh = blockIdx.y, b = blockIdx.z;
  const int split = a.nsplit + ts;
  const int tid = threadIdx.x;
  const int R = a.rep;
  __shared__ float t_q[MAX_REP][D];
  __shared__ float t_P[MAX_REP][32];
  __shared__ float t_alpha[MAX_REP];
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

// Merge of the split partials: out = sum_i o_i 2^{m_i - M} / sum_i l_i 2^{m_i - M}.
// grid (Hq, B), block 256 = 32 channel quads x 8 slices of the list of parts.  What takes time is
// latency - the launch, one round trip to memory, the reduction - so up to 8 MAXU parts are
// requested before the first is used, 16 bytes of a part per thread (a block of 128 threads that
// held 16 or 32 parts as single floats: 3.6 and 5.4 us, 6.4 at 1792 (sequence, head) rows; of 1024
// threads up to 136 parts: 5.8; this: 3.2, 3.3, 4.6 and 4.6).
template <int MAXU>
__global__ __launch_bounds__(256) void attn_merge_kernel(const float* __restrict__ part_o,
                                                         const float2* __restrict__ part_ml,
                                                         int nparts, int BHq,
                                                         _Float16* __restrict__ out) {
  const int row = blockIdx.y * gridDim.x + blockIdx.x;             // (sequence, query head)
  const int c4 = threadIdx.x & 31, sl = threadIdx.x >> 5;
  __shared__ f4 so[8][32];
  __shared__ float sl_[8], sM[8];
  const f4* po = reinterpret_cast<const f4*>(part_o) + (size_t)row * (D / 4) + c4;
  f4 o = f4{0.f, 0.f, 0.f, 0.f};
  float l = 0.0f, M = -INFINITY;
  // slice sl takes parts sl, sl + 8, ...; its sums are relative to its own running maximum
  for (int i0 = sl; i0 < nparts; i0 += 8 * MAXU) {
    f4 oi[MAXU];
    float2 ml[MAXU];
#pragma unroll
    for (int u = 0; u < MAXU; ++u) {
      const int i = i0 + 8 * u, ii = i < nparts ? i : i0;
      oi[u] = po[(size_t)ii * BHq * (D / 4)];
      ml[u] = part_ml[(size_t)ii * BHq + row];
      if (i >= nparts) ml[u].x = -INFINITY;
    }
    float Mn = M;
#pragma unroll
    for (int u = 0; u < MAXU; ++u) Mn = fmaxf(Mn, ml[u].x);
    const float w0 = M == -INFINITY ? 0.0f : exp2f(M - Mn);
    o *= w0;
    l *= w0;
    M = Mn;
#pragma unroll
    for (int u = 0; u < MAXU; ++u) {
      const float w = ml[u].x == -INFINITY ? 0.0f : exp2f(ml[u].x - M);
      if (w != 0.0f) {                       // an empty part's sums are never looked at
        o += w * oi[u];
        l += w * ml[u].y;
      }
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
      const float w = sM[i] == -INFINITY ? 0.0f : exp2f(sM[i] - Mx);
      acc += w * so[i][c >> 2][c & 3];
      L += w * sl_[i];
    }
    out[(size_t)row * D + c] = (_Float16)(L > 0.0f ? acc / L : 0.0f);
  }
}

// Compute units of the current device, asked once per device. A process with no usable
// device (a size query on a build host) gets the MI355X figure, 256.
static int device_cu_count() {
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

// Number of split-T workgroups per (sequence, KV head).
int attn_num_splits(const Geom& g) {
  if (g.ng == 0) return 0;
  const long long bh = (long long)g.B * g.H;
  // 4 waves per workgroup, each wave walks pairs of groups; two workgroups are resident per
  // compute unit, so aim at one full round of them, and at no less than 8 pairs per workgroup
  const long long target = 2LL * device_cu_count();
  long long n = (target + bh - 1) / bh;
  const long long units = ((g.ng + 1) / 2 + 7) / 8;
  if (n > units) n = units;
  if (n < 1) n = 1;
  return (int)n;
}

// A large block of residual tokens is worth a stream of its own: its kernel is short of
// memory parallelism, not of arithmetic, and runs well beside the MFMA kernel.
bool attn_tail_beside(const Geom& g, int cap) {
  if (cap <= 0 || g.ng == 0) return false;
  const int iters = (cap + 31) / 32;
  const long long wgs = (long long)(iters < ATTN_TAIL_SPLITS ? iters : ATTN_TAIL_SPLITS) * g.B * g.H;
  return wgs >= 4LL * device_cu_count();
}

// side / fork / join: when side is not null (and there are residual tokens for the MFMA
// path) the residual-token kernel is forked onto that stream and joined before the merge.
hipError_t launch_decode_attention(const Geom& g, int layer, float scale, const void* q,
                                   const uint8_t* pk, const uint8_t* pv, const void* ktail,
                                   const void* vtail, int cap, const int32_t* tail_len, void* out,
                                   void* ws, unsigned stages, hipStream_t st, hipStream_t side,
                                   hipEvent_t fork, hipEvent_t join) {
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
  a.n_a = g.n_a; a.n_n = g.n_n; a.n_s = g.n_s; a.krec_bytes = g.krec; a.cap = cap;
  a.sal_bits = g.sal_bits; a.npg = g.npg; a.use_fft = g.use_fft ? 1 : 0;
  a.nsplit = attn_num_splits(g);
  a.scale2 = scale * 1.4426950408889634f;
  // stages: bit 0 split-T partial kernel(s), bit 1 merge
  // the residual-token block is a launch of its own, up to ATTN_TAIL_SPLITS workgroups per
  // (sequence, KV head); with no token at all one empty part per head is still written
  const int tail_iters = has_tail ? (cap + 31) / 32 : 0;
  const int ntail = has_tail ? (tail_iters < ATTN_TAIL_SPLITS ? tail_iters : ATTN_TAIL_SPLITS) : (a.nsplit > 0 ? 0 : 1);
  a.tail_per = ntail > 0 && tail_iters > 0 ? (tail_iters + ntail - 1) / ntail : 0;
  const int nparts = a.nsplit + ntail;
  a.part_o = reinterpret_cast<float*>(ws);                        // 16-byte aligned rows
  a.part_ml = a.part_o + (size_t)nparts * g.B * g.Hq * D;
  if (stages & 1u) {
    const int npairs = (g.ng + 1) / 2;
    a.gps = a.nsplit > 0 ? (npairs + a.nsplit - 1) / a.nsplit : 0;   // pairs per split
    const dim3 gtail(ntail, g.H, g.B), gmain(a.nsplit, g.H, g.B);
    if (has_tail && side && a.nsplit > 0) {
      if (hipEventRecord(fork, st) != hipSuccess) return hipErrorUnknown;
      if (hipStreamWaitEvent(side, fork, 0) != hipSuccess) return hipErrorUnknown;
      // the side stream now depends on `st`: it is joined back whatever fails below
      hipLaunchKernelGGL(attn_tail_kernel, gtail, dim3(256), 0, side, a);
      const bool rec = hipEventRecord(join, side) == hipSuccess;
      launch_attn_mfma(a, gmain, st);
      const bool joined = hipStreamWaitEvent(st, join, 0) == hipSuccess;
      if (!rec || !joined) return hipErrorUnknown;
    } else {
      if (a.nsplit > 0) launch_attn_mfma(a, gmain, st);
      if (ntail > 0) hipLaunchKernelGGL(attn_tail_kernel, gtail, dim3(256), 0, st, a);
    }
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
