// Launches of the value coding pass (quant_values_enc.h).
#include "quant_values_enc.h"
#include "select_keys.h"

namespace vidkv {

__global__ __launch_bounds__(256) void v_encode_wave_kernel(
    const u32x4* __restrict__ V, int T, int ng, int B, int H, int n_s, float gamma,
    int gpb, int ngc, int g_out0, const uint32_t* __restrict__ mask, const uint32_t* __restrict__ rank,
    uint8_t* __restrict__ rec_out, u32x4* __restrict__ rows_out) {
  __shared__ EncTile tile4[4];
  v_encode_part<false>(V, T, ng, B, H, n_s, gamma, gpb, ngc, g_out0, mask, rank, rec_out, rows_out, nullptr, nullptr, -1, blockIdx.x,
                       blockIdx.y, tile4);
}

// The same with the channel selection of the keys of the same call in the first workgroups (rows
// y < sel_rows of the grid): as a launch of its own between the two key passes it cost
// 6 to 8 us in which nothing else ran; here the pass takes as long as without it (33.6 us at 28 x 6272
// tokens, 33.4 before).
// FEW: the selection has left RANK and IDX to this pass.
template <bool FEW>
__global__ __launch_bounds__(256) void v_encode_select_kernel(
    const u32x4* __restrict__ V, int T, int ng, int B, int H, int n_s, float gamma,
    int gpb, int ngc, int g_out0, const uint32_t* __restrict__ mask, uint32_t* __restrict__ rank, int32_t* __restrict__ idx,
    uint8_t* __restrict__ rec_out, u32x4* __restrict__ rows_out, int sel_rows, int heads,
    const _Float16* __restrict__ ws, int chunks, int n_a, uint8_t* __restrict__ perm) {
  __shared__ union { EncTile tile4[4]; ChanSelLds<256> sel; } lds;
  if ((int)blockIdx.y < sel_rows) {
    const int hd = blockIdx.y * gridDim.x + blockIdx.x;
    if (hd < heads) select_channels<256>(ws, chunks, n_a, perm, hd, lds.sel);
    return;
  }
  v_encode_part<false, false, FEW>(V, T, ng, B, H, n_s, gamma, gpb, ngc, g_out0, mask, rank, rec_out, rows_out, nullptr, rank, -1, blockIdx.x,
                       blockIdx.y - sel_rows, lds.tile4, idx);
}

VEncArgs v_encode_args(const Geom& g, const EncodeSpan& sp, int n_s, float gamma, const void* V, uint8_t* packed) {
  // one group per wave: many short-lived workgroups balance the memory system best here
  return VEncArgs{reinterpret_cast<const u32x4*>(V), sp.in_tokens, sp.ng, g.B, g.H, n_s, gamma, 4, g.ngc, sp.g_out0,
                  reinterpret_cast<uint32_t*>(packed + g.v_mask), reinterpret_cast<uint32_t*>(packed + g.v_rank),
                  packed + g.v_rec + (size_t)sp.head0 * g.ngc * VREC,
                  g.sal_bits == 16 ? reinterpret_cast<u32x4*>(packed + g.v_rows) : nullptr, -1, nullptr, 0, nullptr};
}

void launch_v_encode(const Geom& g, const EncodeSpan& sp, int n_s, float gamma, const void* V,
                     uint8_t* packed, hipStream_t st) {
  const VEncArgs a = v_encode_args(g, sp, n_s, gamma, V, packed);
  hipLaunchKernelGGL(v_encode_wave_kernel, dim3((sp.ng + a.gpb - 1) / a.gpb, (unsigned)sp.heads), dim3(256), 0, st,
                     a.V, a.T, a.ng, a.B, a.H, a.n_s, a.gamma, a.gpb, a.ngc,
                     a.g_out0, a.mask, a.rank, a.rec_out, a.rows_out);
}

// Whether the value coding of all heads and their channel selection fit one grid.
bool v_encode_select_fits(const Geom& g) {
  const long long gx = (g.ng + 3) / 4;
  return g.nheads + (g.nheads + gx - 1) / gx <= 65535;
}

// ws: the range pass's partials of the same heads.  few: RANK and IDX are not there yet.
void launch_v_encode_select(const Geom& g, float gamma, const void* V, uint8_t* packed_V, const void* ws,
                            uint8_t* packed_K, bool few, hipStream_t st) {
  const VEncArgs a = v_encode_args(g, EncodeSpan{g.T, g.ng, 0, g.nheads, 0}, g.n_s, gamma, V, packed_V);
  const long long gx = (g.ng + a.gpb - 1) / a.gpb, rows = (g.nheads + gx - 1) / gx;
  auto* kernel = few ? v_encode_select_kernel<true> : v_encode_select_kernel<false>;
  hipLaunchKernelGGL(kernel, dim3((unsigned)gx, (unsigned)(g.nheads + rows)), dim3(256), 0, st,
                     a.V, a.T, a.ng, a.B, a.H, a.n_s, a.gamma, a.gpb, a.ngc,
                     a.g_out0, a.mask, a.rank, reinterpret_cast<int32_t*>(packed_V + g.v_idx), a.rec_out, a.rows_out, (int)rows,
                     (int)g.nheads, reinterpret_cast<const _Float16*>(ws), g.range_chunks, g.n_a, packed_K + g.k_perm);
}

}  // namespace vidkv
