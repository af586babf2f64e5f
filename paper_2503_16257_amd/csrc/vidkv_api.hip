// C ABI of the VidKV library: argument validation on the host, then kernel
// launches on the caller's stream (and, for vidkv_quantize_kv, on a second stream that the
// caller hands in).  Nothing here allocates, synchronizes, or creates streams or events.
#include <mutex>

#include "vidkv_common.h"

namespace vidkv {
hipError_t launch_quantize_keys(const Geom& g, const void* K, uint8_t* packed, void* ws,
                                unsigned stages, hipStream_t st);
hipError_t launch_quantize_values(const Geom& g, float gamma, const void* V, const float* scores,
                                  const int32_t* idx, uint8_t* packed, void* ws,
                                  unsigned stages, hipStream_t st);
size_t values_ws_bytes(const Geom& g);
hipError_t launch_decode_attention(const Geom& g, int layer, float scale, const void* q,
                                   const uint8_t* pk, const uint8_t* pv, const void* ktail,
                                   const void* vtail, int cap, const int32_t* tail_len, void* out,
                                   void* ws, size_t ws_bytes, unsigned stages, hipStream_t st);
int attn_least_splits(const Geom& g);
int attn_max_splits(const Geom& g);
void launch_k_encode(const Geom& g, const EncodeSpan& sp, const void* K, uint8_t* packed,
                     bool use_fft, hipStream_t st);
void launch_v_encode(const Geom& g, const EncodeSpan& sp, int n_s, float gamma, const void* V,
                     uint8_t* packed, hipStream_t st);
bool one_workgroup_selection(const Geom& g);
void launch_k_range_select(const Geom& g, const void* K, void* ws, const float* scores, const int32_t* idx,
                           uint8_t* packed_V, bool few, hipStream_t st);
bool few_selection(const Geom& g, bool scores, bool alone);
bool v_encode_select_fits(const Geom& g);
void launch_v_encode_select(const Geom& g, float gamma, const void* V, uint8_t* packed_V, const void* ws,
                            uint8_t* packed_K, bool few, hipStream_t st);
bool launch_few_groups(const Geom& g, float gamma, const void* K, const void* V, void* ws, const float* scores,
                       const int32_t* idx, uint8_t* packed_K, uint8_t* packed_V, hipStream_t st);
bool launch_k_encode_protect2(const Geom& g, const void* K, uint8_t* packed_K, const void* V, uint8_t* packed_V,
                              hipStream_t st);
void launch_v_protect2(const Geom& g, const void* V, uint8_t* packed, hipStream_t st);
bool launch_flush_encode(const Geom& g, const EncodeSpan& sp, float gamma, const void* K, const void* V,
                         uint8_t* packed_K, uint8_t* packed_V, hipStream_t st);
void launch_flush_marks(const Geom& g, int n_groups, uint8_t* packed, hipStream_t st);
hipError_t launch_saliency(const void* Xv, const void* Xt, int B, int Tv, int Nt, int d,
                           float* scores, float* tsum, hipStream_t st);

static size_t ws_keys(const Geom& g) {
  if (g.metric != 0)     // float64 partials and thresholds of the variance / outlier metrics
    return align256(((size_t)g.nheads * g.range_chunks * 2 + (size_t)g.nheads) * D * sizeof(double)) + 256;
  return align256((size_t)g.nheads * g.range_chunks * 2 * D * sizeof(_Float16)) + 256;
}
static size_t ws_values(const Geom& g) { return values_ws_bytes(g); }
static size_t ws_attn(const Geom& g, int (*splits)(const Geom&) = attn_max_splits) {
  // sized for the capacity, so that a workspace allocated once stays large enough
  // while residual flushes make the packed cache longer
  Geom c = g;
  c.T = g.Tcap;
  c.ng = g.ngc;
  return align256((size_t)(splits(c) + ATTN_TAIL_SPLITS) * g.B * g.Hq * (D + 2) * sizeof(float)) + 256;
}
static bool aligned(const void* p, size_t a) { return (reinterpret_cast<uintptr_t>(p) & (a - 1)) == 0; }

__global__ __launch_bounds__(256) void calib_copy_kernel(const u32x4* __restrict__ src,
                                                         u32x4* __restrict__ dst, size_t n) {
  size_t i = (size_t)blockIdx.x * 1024 + threadIdx.x;
#pragma unroll
  for (int k = 0; k < 4; ++k, i += 256)
    if (i < n) __builtin_nontemporal_store(__builtin_nontemporal_load(src + i), dst + i);
}
}  // namespace vidkv

using namespace vidkv;

namespace {
constexpr int MAX_DEVICES = 64;

// The caller's side stream and events, or nothing.  All three handles must be there.
struct Side {
  hipStream_t stream = nullptr;
  hipEvent_t fork = nullptr, join = nullptr;
  bool ok = false;
};
Side take_side(const vidkv_side_stream* s) {
  Side r;
  if (s && s->hip_stream && s->fork_event && s->join_event) {
    r.stream = static_cast<hipStream_t>(s->hip_stream);
    r.fork = static_cast<hipEvent_t>(s->fork_event);
    r.join = static_cast<hipEvent_t>(s->join_event);
    r.ok = true;
  }
  return r;
}
bool side_malformed(const vidkv_side_stream* s) {
  return s && !(s->hip_stream && s->fork_event && s->join_event);
}

// A stream of another device than the current one cannot take this call's launches.
// (The NULL stream belongs to the current device.  If the runtime cannot tell, go on.)
bool stream_on_current_device(hipStream_t st) {
  if (!st) return true;
  int cur = 0, dev = 0;
  if (hipGetDevice(&cur) != hipSuccess || hipStreamGetDevice(st, &dev) != hipSuccess) {
    (void)hipGetLastError();
    return true;
  }
  return cur == dev;
}
}  // namespace

extern "C" {

size_t vidkv_packed_keys_bytes(const vidkv_params* p) {
  Geom g;
  return make_geom(p, &g) ? g.k_total : 0;
}

size_t vidkv_packed_values_bytes(const vidkv_params* p) {
  Geom g;
  return make_geom(p, &g) ? g.v_total : 0;
}

size_t vidkv_workspace_bytes(const vidkv_params* p, int which) {
  Geom g;
  if (!make_geom(p, &g)) return 0;
  switch (which) {
    case 0: return ws_keys(g);
    case 1: return ws_values(g);
    case 2: return ws_attn(g);
    case 3: return ws_keys(g) + ws_values(g);
    default: return 0;
  }
}

vidkv_status vidkv_quantize_keys_stages(const vidkv_params* p, const void* K, void* packed,
                                        size_t packed_bytes, void* ws, size_t ws_bytes,
                                        uint32_t stages, void* stream) {
  Geom g;
  if (!p || !packed || !ws) return VIDKV_EINVAL;
  if (!make_geom(p, &g)) return VIDKV_ESHAPE;
  if (g.T > 0 && !K) return VIDKV_EINVAL;
  if (g.nheads > 65535) return VIDKV_ESHAPE;
  if (!aligned(K, 16) || !aligned(packed, 256) || !aligned(ws, 256)) return VIDKV_EINVAL;
  if (packed_bytes < g.k_total || ws_bytes < ws_keys(g)) return VIDKV_ENOSPACE;
  const hipError_t e = launch_quantize_keys(g, K, static_cast<uint8_t*>(packed), ws, stages,
                                            static_cast<hipStream_t>(stream));
  return e == hipSuccess ? VIDKV_OK : VIDKV_EHIP;
}

vidkv_status vidkv_quantize_keys(const vidkv_params* p, const void* K, void* packed,
                                 size_t packed_bytes, void* ws, size_t ws_bytes, void* stream) {
  return vidkv_quantize_keys_stages(p, K, packed, packed_bytes, ws, ws_bytes, ~0u, stream);
}

vidkv_status vidkv_quantize_values_stages(const vidkv_params* p, const void* V,
                                          const float* saliency, const int32_t* salient_idx,
                                          void* packed, size_t packed_bytes, void* ws,
                                          size_t ws_bytes, uint32_t stages, void* stream) {
  Geom g;
  if (!p || !packed || !ws) return VIDKV_EINVAL;
  if (!make_geom(p, &g)) return VIDKV_ESHAPE;
  if (g.T > 0 && !V) return VIDKV_EINVAL;
  if (g.nheads > 65535) return VIDKV_ESHAPE;
  if (g.n_s > 0 && ((saliency != nullptr) == (salient_idx != nullptr))) return VIDKV_EINVAL;
  if (!(p->gamma >= 0.0f) || !(p->gamma < 1e30f)) return VIDKV_EINVAL;
  if (!aligned(V, 16) || !aligned(packed, 256) || !aligned(ws, 256) || !aligned(saliency, 16) ||
      !aligned(salient_idx, 4))
    return VIDKV_EINVAL;
  if (packed_bytes < g.v_total || ws_bytes < ws_values(g)) return VIDKV_ENOSPACE;
  const hipError_t e =
      launch_quantize_values(g, p->gamma, V, g.n_s > 0 ? saliency : nullptr,
                             g.n_s > 0 ? salient_idx : nullptr, static_cast<uint8_t*>(packed), ws,
                             stages, static_cast<hipStream_t>(stream));
  return e == hipSuccess ? VIDKV_OK : VIDKV_EHIP;
}

vidkv_status vidkv_quantize_values(const vidkv_params* p, const void* V, const float* saliency,
                                   const int32_t* salient_idx, void* packed, size_t packed_bytes,
                                   void* ws, size_t ws_bytes, void* stream) {
  return vidkv_quantize_values_stages(p, V, saliency, salient_idx, packed, packed_bytes, ws,
                                      ws_bytes, ~0u, stream);
}

vidkv_status vidkv_quantize_kv(const vidkv_params* p, const void* K, const void* V,
                               const float* saliency, const int32_t* salient_idx, void* packed_K,
                               size_t packed_K_bytes, void* packed_V, size_t packed_V_bytes,
                               void* ws, size_t ws_bytes, void* stream,
                               const vidkv_side_stream* side) {
  Geom g;
  if (!p || !packed_K || !packed_V || !ws || side_malformed(side)) return VIDKV_EINVAL;
  if (!make_geom(p, &g)) return VIDKV_ESHAPE;
  if (g.T > 0 && (!K || !V)) return VIDKV_EINVAL;
  if (g.nheads > 65535) return VIDKV_ESHAPE;
  if (g.n_s > 0 && ((saliency != nullptr) == (salient_idx != nullptr))) return VIDKV_EINVAL;
  if (!(p->gamma >= 0.0f) || !(p->gamma < 1e30f)) return VIDKV_EINVAL;
  if (!aligned(K, 16) || !aligned(V, 16) || !aligned(packed_K, 256) || !aligned(packed_V, 256) ||
      !aligned(ws, 256) || !aligned(saliency, 16) || !aligned(salient_idx, 4))
    return VIDKV_EINVAL;
  if (packed_K_bytes < g.k_total || packed_V_bytes < g.v_total) return VIDKV_ENOSPACE;
  if (ws_bytes < ws_keys(g) + ws_values(g)) return VIDKV_ENOSPACE;
  hipStream_t st = static_cast<hipStream_t>(stream);
  uint8_t* pk = static_cast<uint8_t*>(packed_K);
  uint8_t* pv = static_cast<uint8_t*>(packed_V);
  void* ws_k = ws;
  void* ws_v = static_cast<uint8_t*>(ws) + ws_keys(g);
  const float* sc = g.n_s > 0 ? saliency : nullptr;
  const int32_t* ix = g.n_s > 0 ? salient_idx : nullptr;
  if (!stream_on_current_device(st)) return VIDKV_EINVAL;
  if (g.T == 0) return VIDKV_OK;
  // Launches of the whole call: range pass and protected-token selection | value coding and channel
  // selection | key coding and 2-bit protected rows.  The selections are short chains of dependent
  // work that wait for memory, the passes need its bandwidth: a selection in the first workgroups of
  // a pass costs nothing, as launches of its own one of 5 to 8 us (channels) and six of 3 to 5 us
  // (tokens) with the passes waiting (28 x 4 heads of 6272 tokens with 2-bit rows 139 -> 110 us, 64 x 4 heads of 25088 945 -> 912;
  // 105 and 873 now).  Few groups: two launches (launch_few_groups(): one head of 1568 tokens 38.5 -> 19.3 as three, 10.5 so).
  // A sequence too long for one workgroup's registers keeps the chain of six.  With a side stream,
  // and key passes long enough to hide the fork and join, it runs beside them, the value
  // pass last; beside the range pass alone it is the longer of the two (196000 tokens: 154 us
  // against 137).  The line is at 96 MiB of keys: whole calls in line and beside, us, 5 % protected, K and V just written, on two
  // cards: 41 MB 56 and 73, 67 MB 68 to 73 and 74, 101 MB 85 to 92 and 82 to 87, 117 MB 95 to 101 and 88 to 90, 134 MB 102 to 108 and 96 to
  // 100, 164 MB 117 to 124 and 109 to 114, 201 MB 136 to 144 and 128, 268 MB 175 to 180 and 168, 403 MB 244 and 237, 819 MB 463
  // to 469 and 456; of 32 shapes from there on, 1 to 16 sequences, on the same buffers, rotating or just written ones, none above 1.014.
  const bool sel = g.n_s > 0, one = sel && one_workgroup_selection(g);
  const Side sd = take_side(side);
  const size_t key_bytes = (size_t)g.nheads * g.T * D * 2;
  const bool fork = sel && !one && sd.ok && key_bytes >= ((size_t)96 << 20);
  if (fork) {
    if (!stream_on_current_device(sd.stream)) return VIDKV_EINVAL;
    if (hipEventRecord(sd.fork, st) != hipSuccess) return VIDKV_EHIP;
    if (hipStreamWaitEvent(sd.stream, sd.fork, 0) != hipSuccess) return VIDKV_EHIP;
    // from here on the side stream depends on `st`: whatever fails, it is joined back, so
    // that a stream capture on `st` can still be ended
    bool good = launch_quantize_values(g, p->gamma, V, sc, ix, pv, ws_v, 1u, sd.stream) == hipSuccess;
    good = (hipEventRecord(sd.join, sd.stream) == hipSuccess) && good;
    good = good && launch_quantize_keys(g, K, pk, ws_k, ~0u, st) == hipSuccess;
    good = (hipStreamWaitEvent(st, sd.join, 0) == hipSuccess) && good;
    if (!good) return VIDKV_EHIP;
    return launch_quantize_values(g, p->gamma, V, sc, ix, pv, ws_v, 2u, st) == hipSuccess
               ? VIDKV_OK : VIDKV_EHIP;
  }
  if (g.metric == 0 && launch_few_groups(g, p->gamma, K, V, ws_k, sc, ix, pk, pv, st))
    return hipGetLastError() == hipSuccess ? VIDKV_OK : VIDKV_EHIP;
  bool good = true;
  const bool fits = v_encode_select_fits(g), together = g.metric == 0 && one;
  const bool few = together && fits && few_selection(g, sc != nullptr, false);
  if (together) {
    launch_k_range_select(g, K, ws_k, sc, ix, pv, few, st);
  } else {
    if (sel) good = launch_quantize_values(g, p->gamma, V, sc, ix, pv, ws_v, 1u, st) == hipSuccess;
    good = launch_quantize_keys(g, K, pk, ws_k, g.metric == 0 ? 1u : 3u, st) == hipSuccess && good;
  }
  if (!good) return VIDKV_EHIP;
  const EncodeSpan all{g.T, g.ng, 0, g.nheads, 0};
  if (g.metric == 0 && fits) {
    launch_v_encode_select(g, p->gamma, V, pv, ws_k, pk, few, st);
  } else {
    if (g.metric == 0) good = launch_quantize_keys(g, K, pk, ws_k, 2u, st) == hipSuccess;
    launch_v_encode(g, all, g.n_s, p->gamma, V, pv, st);
  }
  const bool rows2 = sel && g.sal_bits == 2;
  if (!rows2 || !launch_k_encode_protect2(g, K, pk, V, pv, st)) {
    launch_k_encode(g, all, K, pk, g.use_fft, st);
    if (rows2) launch_v_protect2(g, V, pv, st);
  }
  return hipGetLastError() == hipSuccess && good ? VIDKV_OK : VIDKV_EHIP;
}

// Argument checks of a decode step, shared by the entry points below.
static vidkv_status check_decode(const vidkv_params* p, Geom* g, int32_t layer, const void* q,
                                 const void* packed_K, const void* packed_V, const void* K_tail,
                                 const void* V_tail, int32_t tail_capacity,
                                 const int32_t* tail_len, const void* out) {
  if (!p || !q || !out) return VIDKV_EINVAL;
  if (!make_geom(p, g)) return VIDKV_ESHAPE;
  if (layer < 0 || layer >= g->L) return VIDKV_EINVAL;
  if (g->T > 0 && (!packed_K || !packed_V)) return VIDKV_EINVAL;
  if (tail_capacity < 0) return VIDKV_EINVAL;
  if (tail_capacity > 0 && tail_len && (!K_tail || !V_tail)) return VIDKV_EINVAL;
  if (g->B > 65535 || g->H > 65535) return VIDKV_ESHAPE;
  if (!(p->softmax_scale > 0.0f) || !(p->softmax_scale < 1e30f)) return VIDKV_EINVAL;
  if (!aligned(q, 16) || !aligned(out, 16) || !aligned(packed_K, 256) || !aligned(packed_V, 256) ||
      !aligned(K_tail, 16) || !aligned(V_tail, 16) || !aligned(tail_len, 4))
    return VIDKV_EINVAL;
  return VIDKV_OK;
}

vidkv_status vidkv_decode_attention_stages(const vidkv_params* p, int32_t layer, const void* q,
                                           const void* packed_K, const void* packed_V,
                                           const void* K_tail, const void* V_tail,
                                           int32_t tail_capacity, const int32_t* tail_len,
                                           void* out, void* ws, size_t ws_bytes, uint32_t stages,
                                           void* stream, const vidkv_side_stream* side) {
  Geom g;
  if (!ws || side_malformed(side)) return VIDKV_EINVAL;
  const vidkv_status chk = check_decode(p, &g, layer, q, packed_K, packed_V, K_tail, V_tail,
                                        tail_capacity, tail_len, out);
  if (chk != VIDKV_OK) return chk;
  if (!aligned(ws, 256)) return VIDKV_EINVAL;
  // ws_attn(g) has room for the finest split; a workspace of the size that this call asked for when it only
  // knew the coarsest is taken as before, and the split fits it
  if (ws_bytes < ws_attn(g, attn_least_splits)) return VIDKV_ENOSPACE;
  const uint8_t* pk = static_cast<const uint8_t*>(packed_K);
  const uint8_t* pv = static_cast<const uint8_t*>(packed_V);
  hipStream_t st = static_cast<hipStream_t>(stream);
  if (!stream_on_current_device(st)) return VIDKV_EINVAL;
  const hipError_t e = launch_decode_attention(g, layer, p->softmax_scale, q, pk, pv, K_tail, V_tail,
                                               tail_capacity, tail_len, out, ws, ws_bytes, stages, st);
  return e == hipSuccess ? VIDKV_OK : VIDKV_EHIP;
}

vidkv_status vidkv_decode_attention(const vidkv_params* p, int32_t layer, const void* q,
                                    const void* packed_K, const void* packed_V, const void* K_tail,
                                    const void* V_tail, int32_t tail_capacity,
                                    const int32_t* tail_len, void* out, void* ws, size_t ws_bytes,
                                    void* stream, const vidkv_side_stream* side) {
  return vidkv_decode_attention_stages(p, layer, q, packed_K, packed_V, K_tail, V_tail,
                                       tail_capacity, tail_len, out, ws, ws_bytes, ~0u, stream, side);
}

}  // extern "C"

// ---- decode step for callers that cannot allocate -------------------------------------------
// The split partials of a decode step (o, m, l per split, sequence and query head) are the one
// scratch buffer of the decode path.  Here they live in a device array that is part of the
// library's image: every GPU that runs the library holds its own copy, at its own address,
// until the process ends.  The array's name is only a handle on the host; its device address
// is looked up once per device (with that device current) and kept.
static __device__ __align__(256) unsigned char scratch[VIDKV_NOALLOC_SCRATCH_BYTES];

namespace {
void* g_scratch_ptr[MAX_DEVICES];
std::mutex g_scratch_mutex;

// device address of `scratch` on the current device; nullptr on failure
void* scratch_on_current_device() {
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= MAX_DEVICES) return nullptr;
  std::lock_guard<std::mutex> lock(g_scratch_mutex);
  if (!g_scratch_ptr[dev]) {
    void* ptr = nullptr;
    if (hipGetSymbolAddress((void**)&ptr, HIP_SYMBOL(scratch)) != hipSuccess || !ptr) return nullptr;
    g_scratch_ptr[dev] = ptr;
  }
  return g_scratch_ptr[dev];
}
}  // namespace

extern "C" {

vidkv_status vidkv_decode_attention_noalloc(const vidkv_params* p, int32_t layer, const void* q,
                                            const void* packed_K, const void* packed_V,
                                            const void* K_tail, const void* V_tail,
                                            int32_t tail_capacity, const int32_t* tail_len,
                                            void* out, void* stream) {
  Geom g;
  const vidkv_status chk = check_decode(p, &g, layer, q, packed_K, packed_V, K_tail, V_tail,
                                        tail_capacity, tail_len, out);
  if (chk != VIDKV_OK) return chk;
  if (ws_attn(g) > (size_t)VIDKV_NOALLOC_SCRATCH_BYTES) return VIDKV_ENOSPACE;
  void* ws = scratch_on_current_device();
  if (!ws) return VIDKV_EHIP;
  if (!stream_on_current_device(static_cast<hipStream_t>(stream))) return VIDKV_EINVAL;
  // Everything runs in line on the caller's stream.  Nothing in the array has to start at zero: the merge reads
  // only the parts that this call's kernels wrote before it.
  const hipError_t e = launch_decode_attention(
      g, layer, p->softmax_scale, q, static_cast<const uint8_t*>(packed_K),
      static_cast<const uint8_t*>(packed_V), K_tail, V_tail, tail_capacity, tail_len, out, ws,
      VIDKV_NOALLOC_SCRATCH_BYTES, ~0u,
      static_cast<hipStream_t>(stream));
  return e == hipSuccess ? VIDKV_OK : VIDKV_EHIP;
}

vidkv_status vidkv_flush_residual(const vidkv_params* p, int32_t layer, const void* K_tail,
                                  const void* V_tail, int32_t tail_capacity, int32_t n_flush,
                                  void* packed_K, size_t packed_K_bytes, void* packed_V,
                                  size_t packed_V_bytes, void* stream) {
  Geom g;
  if (!p || !K_tail || !V_tail || !packed_K || !packed_V) return VIDKV_EINVAL;
  if (!make_geom(p, &g)) return VIDKV_ESHAPE;
  if (layer < 0 || layer >= g.L) return VIDKV_EINVAL;
  if (n_flush <= 0 || n_flush % G || tail_capacity < n_flush) return VIDKV_EINVAL;
  if (g.T == 0) return VIDKV_EINVAL;               // no channel selection to code the keys with
  if (!(p->gamma >= 0.0f) || !(p->gamma < 1e30f)) return VIDKV_EINVAL;
  if ((long long)g.B * g.H > 65535) return VIDKV_ESHAPE;
  if (!aligned(K_tail, 16) || !aligned(V_tail, 16) || !aligned(packed_K, 256) ||
      !aligned(packed_V, 256))
    return VIDKV_EINVAL;
  if (g.T + n_flush > g.Tcap) return VIDKV_ENOSPACE;
  if (packed_K_bytes < g.k_total || packed_V_bytes < g.v_total) return VIDKV_ENOSPACE;
  hipStream_t st = static_cast<hipStream_t>(stream);
  const long long bh = (long long)g.B * g.H;
  const EncodeSpan sp{tail_capacity, n_flush / G, g.ng, bh, layer * bh};
  uint8_t* pk = static_cast<uint8_t*>(packed_K);
  uint8_t* pv = static_cast<uint8_t*>(packed_V);
  if (!launch_flush_encode(g, sp, p->gamma, K_tail, V_tail, pk, pv, st)) {
    launch_k_encode(g, sp, K_tail, pk, g.use_fft, st);
    launch_v_encode(g, sp, 0, p->gamma, V_tail, pv, st);
    launch_flush_marks(g, sp.ng, pv, st);
  }
  return hipGetLastError() == hipSuccess ? VIDKV_OK : VIDKV_EHIP;
}

size_t vidkv_saliency_workspace_bytes(int32_t batch, int32_t hidden_dim) {
  if (batch < 1 || hidden_dim < 8) return 0;
  return align256((size_t)batch * hidden_dim * sizeof(float));
}

vidkv_status vidkv_saliency_scores(const void* X_v, const void* X_t, int32_t batch,
                                   int32_t n_visual, int32_t n_text, int32_t hidden_dim,
                                   float* scores, void* ws, size_t ws_bytes, void* stream) {
  if (!X_t || !ws) return VIDKV_EINVAL;
  if (batch < 1 || n_visual < 0 || n_text < 1) return VIDKV_EINVAL;
  if (n_visual > 0 && (!X_v || !scores)) return VIDKV_EINVAL;
  if (hidden_dim < 8 || hidden_dim % 8 || hidden_dim > 16384 || batch > 65535) return VIDKV_ESHAPE;
  if (!aligned(X_v, 16) || !aligned(X_t, 2) || !aligned(scores, 4) || !aligned(ws, 256))
    return VIDKV_EINVAL;
  if (ws_bytes < vidkv_saliency_workspace_bytes(batch, hidden_dim)) return VIDKV_ENOSPACE;
  const hipError_t e = launch_saliency(X_v, X_t, batch, n_visual, n_text, hidden_dim, scores,
                                       static_cast<float*>(ws), static_cast<hipStream_t>(stream));
  return e == hipSuccess ? VIDKV_OK : VIDKV_EHIP;
}

vidkv_status vidkv_calib_copy(void* dst, const void* src, size_t bytes, void* stream) {
  if (!dst || !src) return VIDKV_EINVAL;
  if (bytes % 16 || !aligned(dst, 16) || !aligned(src, 16)) return VIDKV_EINVAL;
  if (bytes == 0) return VIDKV_OK;
  const size_t n = bytes / 16;
  const size_t blocks = (n + 1023) / 1024;
  if (blocks > 0x7fffffffull) return VIDKV_ESHAPE;
  hipLaunchKernelGGL(calib_copy_kernel, dim3((unsigned)blocks), dim3(256), 0,
                     static_cast<hipStream_t>(stream), static_cast<const u32x4*>(src),
                     static_cast<u32x4*>(dst), n);
  return hipGetLastError() == hipSuccess ? VIDKV_OK : VIDKV_EHIP;
}

const char* vidkv_status_string(vidkv_status s) {
  switch (s) {
    case VIDKV_OK: return "ok";
    case VIDKV_EINVAL: return "invalid argument";
    case VIDKV_ESHAPE: return "unsupported shape";
    case VIDKV_ENOSPACE: return "buffer too small";
    case VIDKV_EHIP: return "HIP runtime error";
    default: return "unknown status";
  }
}

int vidkv_abi_version(void) { return VIDKV_ABI_VERSION; }

}  // extern "C"
