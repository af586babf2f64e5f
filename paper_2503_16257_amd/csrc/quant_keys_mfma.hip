// Key coding pass (Alg. 3): per 32-token group the 2-bit uniform code (Eq. 4)
// of the anomalous channels and the FFT-based 1-bit code (Eq. 5) of the others.
//
// The 32-point DFT along the tokens is a dense contraction, so it runs on
// v_mfma_f32_16x16x32_f16.  One wave codes one group at a time:
//  1. The [32 tokens x 128 channels] fp16 tile goes global -> registers -> LDS
//     with 16-byte accesses (rows padded to 272 bytes).
//  2. Each lane reads, for a tile of 16 channels taken from the head's channel
//     permutation, its channel at its 8 token slots with 16-bit LDS loads that
//     fill register halves directly: the MFMA operand of a contraction over
//     tokens, gathered and transposed for free.
//  3. Normal channels: the DFT matrix, split in three fp16 parts (exact products,
//     fp32 accumulation), times X (32 tokens x 16 channels), as [slot][channel]:
//     each lane gets 8 coefficients of one channel, so the mean-|.| scales need
//     only a 4-lane sum, and the 8 channels' signs of a slot, a byte of the
//     record's sign words, are or-ed together by register moves between lanes.  One
//     orientation serves both: a second one for the sign bits cost 40 % more MFMA work.
//  4. Anomalous channels: min / max over the 32 tokens, codes, 4 channels per
//     byte assembled inside lane quads.
// The record is assembled in LDS and written with 16-byte stores.
#include "protect2.h"
#include "quant_values_enc.h"
#include "select_keys.h"

namespace vidkv {

constexpr int ENC_MAXT = 9;          // channel tiles of 16: at most 1 + 8
constexpr int ENC_ROW = VENC_ROW;    // LDS bytes per token row (256 + 16 of padding)

// DFT operand table.  Slot x of tile tt (tt = 0: Re X[0..15]; tt = 1: Re X[16],
// Im X[1..15]) against token t: 64 * (w/2) * {cos, -sin}(2 pi k t / 32), with
// w = 1 for the two real-only bins and 2 otherwise, so that the sum of |D| over
// a channel's slots is 1024 * Mean|.| of Eq. 5; positive row scaling does not
// change a sign.  Each fp32 entry is split into three fp16 parts that add up to
// it exactly.  Indexed [tt][part][lane][4 words]: the 8 halves of a lane's
// MFMA operand (slot x = lane & 15, tokens slot_token(lane >> 4, 0..7)).
struct DftTab { uint32_t w[2][3][64][4]; };

constexpr uint32_t half_bits(_Float16 h) { return __builtin_bit_cast(uint16_t, h); }

constexpr DftTab make_dft_tab() {
  DftTab tab{};
  for (int tt = 0; tt < 2; ++tt)
    for (int lane = 0; lane < 64; ++lane)
      for (int i = 0; i < 8; ++i) {
        const int kb = lane >> 4, k = lane & 15;
        const int t = (i < 4) ? 4 * kb + i : 16 + 4 * kb + (i - 4);
        float w = 0.0f;
        if (tt == 0) w = cos32(k * t) * (k == 0 ? 32.0f : 64.0f);
        else         w = (k == 0) ? ((t & 1) ? -32.0f : 32.0f) : -cos32(k * t + 24) * 64.0f;
        if (w == 0.0f) w = 0.0f;                       // no negative zero
        const _Float16 a = (_Float16)w;
        const float r1 = w - (float)a;
        const _Float16 b = (_Float16)r1;
        const _Float16 c = (_Float16)(r1 - (float)b);
        const int sh = 16 * (i & 1);
        tab.w[tt][0][lane][i >> 1] |= half_bits(a) << sh;
        tab.w[tt][1][lane][i >> 1] |= half_bits(b) << sh;
        tab.w[tt][2][lane][i >> 1] |= half_bits(c) << sh;
      }
  return tab;
}

static __device__ const DftTab kDftTab = make_dft_tab();

// v | v of the lane that DPP control CTRL names (one instruction)
template <int CTRL>
__device__ __forceinline__ uint32_t or_dpp(uint32_t v) {
  return v | (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, 0xF, 0xF, true);
}
constexpr int DPP_XOR1 = 0xB1, DPP_XOR2 = 0x4E, DPP_HALF_MIRROR = 0x141, DPP_ROR4 = 0x124, DPP_ROR8 = 0x128;
// the sign bits of four floats, bit 7 of four bytes
__device__ __forceinline__ uint32_t signs4(f4 a) {
  const uint32_t lo = __builtin_amdgcn_perm(__float_as_uint(a[1]), __float_as_uint(a[0]), 0x0C0C0703u);
  const uint32_t hi = __builtin_amdgcn_perm(__float_as_uint(a[3]), __float_as_uint(a[2]), 0x07030C0Cu);
  return lo | hi;
}
// The sign words of the two 8-channel blocks of a tile.  lo, hi: my channel's bits at slots 4 kb .. 4 kb + 3 of
// the first and the second slot tile, at bit 7 of a byte each.  Eight lanes' bits are put at their channel's place
// and or-ed together, so that every lane of a block holds the block's bytes; the first writes 8 of them.
// (As wave-wide ballots whose bytes 32 lanes then selected this took 55 vector instructions a tile, 18 so, in a
// pass whose vector units were 71 % busy.)
__device__ __forceinline__ void put_sign_words(uint8_t* words, uint32_t lo, uint32_t hi, int x16, int kb, bool ok) {
  const uint32_t sh = 7u - (x16 & 7);
  lo = or_dpp<DPP_HALF_MIRROR>(or_dpp<DPP_XOR2>(or_dpp<DPP_XOR1>((lo & 0x80808080u) >> sh)));
  hi = or_dpp<DPP_HALF_MIRROR>(or_dpp<DPP_XOR2>(or_dpp<DPP_XOR1>((hi & 0x80808080u) >> sh)));
  asm("" : "+v"(lo), "+v"(hi));                      // (the last "or" stays outside the branch, one instruction with its move)
  if ((x16 & 7) == 0 && ok)
    *reinterpret_cast<uint2*>(words + (x16 >> 3) * 32 + kb * 8) =
        uint2{__builtin_amdgcn_perm(hi, lo, 0x05010400u), __builtin_amdgcn_perm(hi, lo, 0x07030602u)};
}

// lo, nh: min and -max of my column over the 32 tokens, of which X holds 8.  A NaN counts for nothing (a column of
// nothing else: +infinity, both), so that the other tokens are coded as without it and no code leaves its field.
// (Eight more vector instructions a tile than with minima that pass a NaN on: 28 layers x 4 heads x 6272 tokens,
// n_a = 64, whole call: 107.8 us against 107.2; 64 x 4 x 25088, n_a = 32, plain code: 881 against 886.)
__device__ __forceinline__ void range32(const Op& X, float& lo, float& nh) {
  const h2 mn2 = __builtin_elementwise_min(__builtin_elementwise_min(X.p[0], X.p[1]), __builtin_elementwise_min(X.p[2], X.p[3]));
  const h2 mx2 = __builtin_elementwise_max(__builtin_elementwise_max(X.p[0], X.p[1]), __builtin_elementwise_max(X.p[2], X.p[3]));
  // (against infinity: no NaN from here on, so that the minima across lanes need no canonicalisation)
  lo = fminf(fminf((float)mn2[0], (float)mn2[1]), INFINITY);
  nh = fminf(fminf(-(float)mx2[0], -(float)mx2[1]), INFINITY);
  // both are "min" reductions over the 4 lane groups, so one swap pair serves the two values; a last
  // swap hands both to every lane
  auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(lo), __float_as_uint(nh), false, false);
  const float t = __builtin_elementwise_minimum(__uint_as_float(r[0]), __uint_as_float(r[1]));
  auto q = __builtin_amdgcn_permlane16_swap(__float_as_uint(t), __float_as_uint(t), false, false);
  const float u = __builtin_elementwise_minimum(__uint_as_float(q[0]), __uint_as_float(q[1]));   // rows 0,1: min; rows 2,3: -max
  auto w = __builtin_amdgcn_permlane32_swap(__float_as_uint(u), __float_as_uint(u), false, false);
  lo = __uint_as_float(w[0]);
  nh = __uint_as_float(w[1]);
}

// NA8T >= 0 fixes n_a = 8 * NA8T at compile time (tile loop fully unrolled);
// NA8T < 0 takes n_a at run time.  FFT = false codes the normal channels with
// Eq. 4 at 1 bit on the tokens themselves (the non-FFT 1-bit path of Alg. 3):
// the record keeps its shape, bit (blk, k) e / 8 + e holds the code of channel
// 8 blk + e at token k / 16 + k, and the two scale slots hold s = max - min and
// z = min.
// EXTRA: rows of the grid that do something else of the same call, 1: from row x_rows on, code the
// protected value rows (2 bits), 2: the first x_rows, the value coding pass (a flush: both blocks are
// small, one launch), 3: the first x_rows, the value coding pass of a call with few groups, the next as many the keys, whose
// workgroups select their head's channels themselves, then the protected value rows (2 bits).
// SPLIT: one group per workgroup, its tiles shared out among the four waves (and a flush's values likewise), for
// calls that leave compute units idle anyway: a group's tiles one after another are then most of the kernel
// after the first load.  (Whole calls: one head x 1568 tokens 18.4 us, 17.0 so; 28 flushes of 4 heads x 128 tokens 5 %
// less.  The value pass of a prefill shared out likewise gains nothing beside its channel selection.)
template <int NA8T, bool FFT, int EXTRA, bool SPLIT>
__global__ __launch_bounds__(256) void k_encode_mfma_kernel(const u32x4* __restrict__ K,
                                                            const uint8_t* __restrict__ perm_g,
                                                            int T, int ng, int n_a_rt, int krec,
                                                            int ngc, int g_out0,
                                                            uint8_t* __restrict__ rec_out, int x_rows,
                                                            Protect2Args p2, VEncArgs ve) {
  const int n_a = NA8T >= 0 ? 8 * NA8T : n_a_rt;
  __shared__ EncTile tile4[4];                    // per wave: the group's tile
  if (EXTRA == 1 && (int)blockIdx.y >= x_rows) {
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const long long id = 4 * ((long long)(blockIdx.y - x_rows) * gridDim.x + blockIdx.x) + w;
    if (id < p2.total) protect2_part(p2, id, reinterpret_cast<Protect2Lds*>(&tile4[0][0])[w]);
    return;
  }
  if (EXTRA == 2 && (int)blockIdx.y < x_rows) {
    v_encode_part<true, SPLIT>(ve.V, ve.T, ve.ng, ve.B, ve.H, ve.n_s, ve.gamma, ve.gpb, ve.ngc, ve.g_out0, ve.mask, ve.rank,
                        ve.rec_out, ve.rows_out, ve.mask, ve.rank, ve.mark_rank, blockIdx.x, blockIdx.y, tile4);
    return;
  }
  if (EXTRA == 3 && (int)blockIdx.y >= 2 * x_rows) {
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const long long id = 4 * ((long long)(blockIdx.y - 2 * x_rows) * gridDim.x + blockIdx.x) + w;
    if (id < p2.total) protect2_part<true>(p2, id, reinterpret_cast<Protect2Lds*>(&tile4[0][0])[w]);
    return;
  }
  if (EXTRA == 3 && (int)blockIdx.y < x_rows) {
    v_encode_part<false, true, true>(ve.V, ve.T, ve.ng, ve.B, ve.H, ve.n_s, ve.gamma, 1, ve.ngc, 0, ve.mask, ve.rank,
                        ve.rec_out, ve.rows_out, nullptr, ve.rank, -1, blockIdx.x, blockIdx.y, tile4, ve.idx);
    return;
  }
  const long long hd = blockIdx.y - (EXTRA >= 2 ? x_rows : 0);
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int x16 = lane & 15, kb = lane >> 4;
  const int n_n = D - n_a;
  const int NTa = (n_a + 15) >> 4, NTn = (n_n + 15) >> 4, NT = NTa + NTn;
  const int nq = n_a >> 2;

  // per wave: the record being assembled (12 n_a + 8 n_n bytes; 1536 at most).  With n_a known
  // the workgroup stays below a quarter of the LDS and four of them share a compute unit.
  constexpr int RECB = NA8T >= 0 ? 12 * 8 * NA8T + 8 * (D - 8 * NA8T) : 1536;
  __shared__ u32x4 recbuf[4][RECB / 16];

  // the first tile is requested before anything else so that its latency
  // overlaps the set-up below
  const int g = SPLIT ? blockIdx.x : blockIdx.x * 4 + wave;
  if (g >= ng) return;                               // (unless SPLIT there is no barrier below: everything is per wave)
  const int slot = SPLIT ? 0 : wave;                 // which tile and record buffer
  const u32x4* head = K + hd * (long long)T * 16;

  // coalesced tile load: lane reads 16 bytes of row (lane >> 4) + 4 i, i = 0..7
  constexpr int NPRE = SPLIT ? 2 : 8;                // SPLIT: my wave's rows are 8 wave ..
  const int row0 = SPLIT ? 8 * wave : 0;
  u32x4 pre[NPRE];
#pragma unroll
  for (int i = 0; i < NPRE; ++i) pre[i] = __builtin_nontemporal_load(head + ((long long)g * G + row0) * 16 + lane + 64 * i);
  FewChanLds& chan = reinterpret_cast<FewChanLds&>(tile4[1]);
  static_assert(sizeof(FewChanLds) <= 3 * sizeof(EncTile), "beside the one tile that is in use");
  if (EXTRA == 3) {
    few_channels(ve.range_ws, ve.chunks, n_a, g == 0 ? const_cast<uint8_t*>(perm_g) : nullptr, hd, chan);
    __syncthreads();
  }
  __builtin_amdgcn_sched_barrier(0);                 // (these first, and their first use behind the set-up: 1 % of a call with 4 heads x 196000)

  // Channel tile j: anomalous tiles first (16 anomalous channels each, in PERM
  // order), then normal tiles.  My column's channel in every tile, as a byte
  // offset inside a token row (an absent column reads channel 0 and is ignored).
  constexpr int NMY = SPLIT ? (ENC_MAXT + 3) / 4 : ENC_MAXT;
  int chofs[NMY];
#pragma unroll
  for (int jj = 0; jj < NMY; ++jj) {
    const int j = SPLIT ? 4 * jj + wave : jj;
    const bool an = j < NTa;
    const int off = an ? 16 * j + x16 : 16 * (j - NTa) + x16;
    const bool valid = j < NT && (an ? off < n_a : off < n_n);
    const int at = an ? off : n_a + off;
    chofs[jj] = valid ? 2 * (int)(EXTRA == 3 ? chan.perm[at] : perm_g[hd * D + at]) : 0;
  }

  // DFT operand from the precomputed table: slot x16 of tile tt, k-slots = tokens
  Op F[2][3];
  if (FFT) {
#pragma unroll
    for (int tt = 0; tt < 2; ++tt)
#pragma unroll
      for (int part = 0; part < 3; ++part)
        F[tt][part].q = *reinterpret_cast<const u32x4*>(&kDftTab.w[tt][part][lane][0]);
  }

  uint8_t* rec8 = reinterpret_cast<uint8_t*>(&recbuf[slot][0]);
  uint16_t* rec16 = reinterpret_cast<uint16_t*>(rec8);
  const int bits_h = 6 * n_a;                        // half-word offsets inside the record
  const int meta_h = 6 * n_a + 2 * n_n;
  const int nblk = n_n >> 3;
  float one = 1.0f;                                  // (a 1 that the compiler does not see)
  asm("" : "+v"(one));
  // my 8 token slots start at row 4*kb (slots 0-3) and 16 + 4*kb (slots 4-7)
  const uint8_t* tcol = reinterpret_cast<const uint8_t*>(&tile4[slot][0]) + 4 * kb * ENC_ROW;

  __builtin_amdgcn_sched_barrier(0);
  {
    uint8_t* wdst = reinterpret_cast<uint8_t*>(&tile4[slot][0]) + (row0 + kb) * ENC_ROW + x16 * 16;
#pragma unroll
    for (int i = 0; i < NPRE; ++i) *reinterpret_cast<u32x4*>(wdst + 4 * i * ENC_ROW) = pre[i];
  }
  if (SPLIT) __syncthreads();

#pragma unroll
  for (int jj = 0; jj < NMY; ++jj) {
    const int j = SPLIT ? 4 * jj + wave : jj;
    if (j >= NT) break;
    // my column's channel at my 8 token slots: 16-bit LDS loads into register halves
    Op X;
    const uint8_t* cp = tcol + chofs[jj];
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const int row = (i < 4) ? i : 12 + i;          // relative to row 4*kb
      X.v[i] = *reinterpret_cast<const _Float16*>(cp + row * ENC_ROW);
    }

    if (j < NTa) {
      // ---------------- Eq. 4, 2 bits: z = min, s = (max - min) / 3 over the 32 tokens
      float lo_f, nh_f;
      range32(X, lo_f, nh_f);
      const float mnf = lo_f, rng = -nh_f - lo_f;
      const float inv = rng > 0.0f ? 3.0f / rng : 0.0f;
      uint32_t w0 = 0, w1 = 0;
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        // between 0 and a little over 3, whatever the rounding, or a NaN, whose code is 0: nothing to clamp.
        // (x - min as x * 1 + (-min): a multiply-add takes the 16-bit operand as it is)
        const float u = rintf(__builtin_fmaf((float)X.v[i], one, -mnf) * inv);
        if (i < 4) w0 = __builtin_amdgcn_cvt_pk_u8_f32(u, i, w0); else w1 = __builtin_amdgcn_cvt_pk_u8_f32(u, i - 4, w1);
      }
      // 4 channels of a quad (adjacent lanes) share a byte: channel r in bits 2r, 2r+1
      const int ja = 16 * j + x16;                 // anomalous index of my column
      w0 <<= 2 * (x16 & 3);
      w1 <<= 2 * (x16 & 3);
      if (ja >= n_a) { w0 = 0; w1 = 0; }
      w0 = or_dpp<DPP_XOR2>(or_dpp<DPP_XOR1>(w0));
      w1 = or_dpp<DPP_XOR2>(or_dpp<DPP_XOR1>(w1));
      // the quads' bytes of a token are neighbours: lane (quad, r) takes token r's byte to its quad's place, and the
      // four quads' are or-ed (8 single bytes from every fourth lane before)
      const uint32_t to_place = 0x0C0C0C0Cu ^ ((0x0Cu ^ (x16 & 3)) << (2 * (x16 & 12)));
      w0 = or_dpp<DPP_ROR8>(or_dpp<DPP_ROR4>(__builtin_amdgcn_perm(0u, w0, to_place)));
      w1 = or_dpp<DPP_ROR8>(or_dpp<DPP_ROR4>(__builtin_amdgcn_perm(0u, w1, to_place)));
      if (x16 < 8) {                               // quad 0: the first four slots' tokens, quad 1: the others
        uint8_t* at = rec8 + ((x16 & 4 ? 16 : 0) + 4 * kb + (x16 & 3)) * nq + 4 * j;
        const uint32_t v = x16 & 4 ? w1 : w0;
        if ((nq & 3) == 0) {
          *reinterpret_cast<uint32_t*>(at) = v;
        } else {                                   // n_a = 8 mod 16: rows of codes are 2-byte aligned, the last tile half full
          *reinterpret_cast<uint16_t*>(at) = (uint16_t)v;
          if (16 * j + 16 <= n_a) *reinterpret_cast<uint16_t*>(at + 2) = (uint16_t)(v >> 16);
        }
      }
      if (kb == 0 && ja < n_a) {
        // rng / 3, correctly rounded: the product with the rounded 1/3 and one correction
        const float q3 = rng * (1.0f / 3.0f);
        const float s = __builtin_fmaf(__builtin_fmaf(-3.0f, q3, rng), 1.0f / 3.0f, q3);
        reinterpret_cast<_Float16*>(rec16)[4 * n_a + ja] = (_Float16)s;
        reinterpret_cast<_Float16*>(rec16)[5 * n_a + ja] = (_Float16)lo_f;
      }
    } else if (!FFT) {
      // ---------------- Eq. 4, 1 bit: z = min, s = max - min over the 32 tokens
      const int jn = j - NTa;
      float lo_f, nh_f;
      range32(X, lo_f, nh_f);
      const float rng = -nh_f - lo_f;
      // code = round-half-even((x - z) / s) in {0, 1} = [x above the midpoint]; a tie codes 0
      const float mid = 0.5f * (lo_f - nh_f);
      const int nidx = 16 * jn + x16;              // normal index of my column
      // x above the midpoint = x above the largest fp16 number that is not above the midpoint = the sign of their
      // difference.  That number: the midpoint (+ 0: no -0, whose difference to +0 would be negative) rounded
      // toward zero, and where that went up, the next one down
      const float mid0 = mid + 0.0f;
      uint32_t t = __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_pkrtz(mid0, mid0));
      t += (float)bits_h2(t)[0] > mid0 ? 0x00010001u : 0u;
      uint32_t d[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) d[i] = h2_bits(bits_h2(t) - X.p[i]);
      // slots (0, 1), (2, 3): tokens 4 kb + i; slots (4, 5), (6, 7): tokens 16 + 4 kb + i
      put_sign_words(rec8 + 2 * bits_h + 64 * jn, __builtin_amdgcn_perm(d[1], d[0], 0x07050301u),
                     __builtin_amdgcn_perm(d[3], d[2], 0x07050301u), x16, kb, 2 * jn + (x16 >> 3) < nblk);
      if ((kb & 1) == 0 && nidx < n_n) {
        const int b8 = nidx >> 3, e = nidx & 7;
        reinterpret_cast<_Float16*>(rec16)[meta_h + (b8 * 2 + (kb >> 1)) * 8 + e] =
            (kb >> 1) ? (_Float16)lo_f : (_Float16)rng;
      }
    } else {
      // ---------------- Eq. 5: 32-point DFT along tokens, sign bits and mean-|.| scales
      const int jn = j - NTa;
      const f4 zero = f4{0.f, 0.f, 0.f, 0.f};
      // [slot][channel]: my column = channel x16, my rows = slots 4kb + i of the two slot
      // tiles (Re X[0..15]; Re X[16], Im X[1..15]); three exact partial products each
      f4 aRe = mma(F[0][0], X, zero), aIm = mma(F[1][0], X, zero);
      aRe = mma(F[0][1], X, aRe);  aIm = mma(F[1][1], X, aIm);
      aRe = mma(F[0][2], X, aRe);  aIm = mma(F[1][2], X, aIm);
      const int nidx = 16 * jn + x16;              // normal index of my column
      // sign bits (bit = coefficient >= 0; a sum that starts at +0 is never -0)
      put_sign_words(rec8 + 2 * bits_h + 64 * jn, ~signs4(aRe), ~signs4(aIm), x16, kb, 2 * jn + (x16 >> 3) < nblk);
      // scales: Re X[16] sits in row 0 of the second tile and counts for the real view
      float sr = fabsf(aRe[0]) + fabsf(aRe[1]) + fabsf(aRe[2]) + fabsf(aRe[3]);
      float si = fabsf(aIm[0]) + fabsf(aIm[1]) + fabsf(aIm[2]) + fabsf(aIm[3]);
      if (kb == 0) { sr += fabsf(aIm[0]); si -= fabsf(aIm[0]); }
      // sum over the 4 lane groups: afterwards rows 0,1 hold the Re total, rows 2,3 the Im total
      auto r32 = __builtin_amdgcn_permlane32_swap(__float_as_uint(sr), __float_as_uint(si), false, false);
      const float t2 = __uint_as_float(r32[0]) + __uint_as_float(r32[1]);
      auto r16 = __builtin_amdgcn_permlane16_swap(__float_as_uint(t2), __float_as_uint(t2), false, false);
      const float tot = (__uint_as_float(r16[0]) + __uint_as_float(r16[1])) * (1.0f / 1024.0f);
      if ((kb & 1) == 0 && nidx < n_n) {
        const int b8 = nidx >> 3, e = nidx & 7;
        reinterpret_cast<_Float16*>(rec16)[meta_h + (b8 * 2 + (kb >> 1)) * 8 + e] = (_Float16)tot;
      }
    }
  }
  // ---- the finished record: LDS -> global, 16 bytes per lane
  u32x4* dst = reinterpret_cast<u32x4*>(rec_out + (hd * ngc + g_out0 + g) * (long long)krec);
  const int nch = krec >> 4;
  if (SPLIT) {
    __syncthreads();
    if (tid < nch) __builtin_nontemporal_store(recbuf[0][tid], dst + tid);
  } else {
    if (lane < nch) __builtin_nontemporal_store(recbuf[wave][lane], dst + lane);
    if (lane + 64 < nch) __builtin_nontemporal_store(recbuf[wave][lane + 64], dst + lane + 64);
  }
}

template <int NA8T, int EXTRA, bool SPLIT>
static void launch_one(bool use_fft, dim3 grid, hipStream_t st, const u32x4* k4, const uint8_t* perm, const Geom& g,
                       const EncodeSpan& sp, uint8_t* rec, int rows, const Protect2Args& p2, const VEncArgs& ve) {
  if (EXTRA == 1) rows = (int)sp.heads;
  if (use_fft)
    hipLaunchKernelGGL((k_encode_mfma_kernel<NA8T, true, EXTRA, SPLIT>), grid, dim3(256), 0, st, k4, perm, sp.in_tokens, sp.ng,
                       g.n_a, g.krec, g.ngc, sp.g_out0, rec, rows, p2, ve);
  else
    hipLaunchKernelGGL((k_encode_mfma_kernel<NA8T, false, EXTRA, SPLIT>), grid, dim3(256), 0, st, k4, perm, sp.in_tokens, sp.ng,
                       g.n_a, g.krec, g.ngc, sp.g_out0, rec, rows, p2, ve);
}

template <int EXTRA, bool SPLIT>
static void launch_any(const Geom& g, const EncodeSpan& sp, int gx, const void* K, uint8_t* packed, bool use_fft,
                       hipStream_t st, int rows, const Protect2Args& p2, const VEncArgs& ve, int more = 0) {
  const dim3 grid(gx, (unsigned)(sp.heads + rows + more));
  const u32x4* k4 = reinterpret_cast<const u32x4*>(K);
  const uint8_t* perm = packed + g.k_perm + sp.head0 * D;
  uint8_t* rec = packed + g.k_rec + (size_t)sp.head0 * g.ngc * g.krec;
  switch (g.n_a) {
    case 8:  launch_one<1, EXTRA, SPLIT>(use_fft, grid, st, k4, perm, g, sp, rec, rows, p2, ve); break;
    case 16: launch_one<2, EXTRA, SPLIT>(use_fft, grid, st, k4, perm, g, sp, rec, rows, p2, ve); break;
    case 32: launch_one<4, EXTRA, SPLIT>(use_fft, grid, st, k4, perm, g, sp, rec, rows, p2, ve); break;
    case 64: launch_one<8, EXTRA, SPLIT>(use_fft, grid, st, k4, perm, g, sp, rec, rows, p2, ve); break;
    case 0: launch_one<0, EXTRA, SPLIT>(use_fft, grid, st, k4, perm, g, sp, rec, rows, p2, ve); break;
    case 96: launch_one<12, EXTRA, SPLIT>(use_fft, grid, st, k4, perm, g, sp, rec, rows, p2, ve); break;
    case 128: launch_one<16, EXTRA, SPLIT>(use_fft, grid, st, k4, perm, g, sp, rec, rows, p2, ve); break;
    default: launch_one<-1, EXTRA, SPLIT>(use_fft, grid, st, k4, perm, g, sp, rec, rows, p2, ve); break;
  }
}

// Four groups per workgroup, one per wave: short-lived workgroups keep the memory system evenly loaded.  (Two per
// wave, the second's load beside the first's arithmetic, were better while the arithmetic took most of the time.  When
// it no longer did, whole calls on one card: 64 x 4 heads x 25088 tokens, n_a = 32, plain code, 3 % slower than this,
// 4 heads x 196000 2 %, 28 x 4 x 6272, n_a = 64, the same.)
constexpr int K_GPB = 4;

// One group per workgroup, its tiles among the four waves: where no compute unit gets more than one such workgroup.
// (The kernel alone, inputs in the caches, one group per wave against shared out, n_a = 64: 49 groups 4.6 us against 3.1, 128 4.7 against
// 3.3, 200 5.0 against 3.5, 256 5.0 against 3.6, whether of one head or of eight; n_a = 16: 4.6 against 3.4 to 4.9 against 3.6;
// a flush with its values: 32 groups 4.6 against 3.2, 256 4.7 against 3.6.  Beyond the compute units the difference falls:
// 300 groups 5.0 against 3.9, 512 5.2 against 4.2; not looked at in whole calls.)
static bool split_groups(long long groups) { return groups <= device_cu_count(); }

void launch_k_encode(const Geom& g, const EncodeSpan& sp, const void* K, uint8_t* packed,
                     bool use_fft, hipStream_t st) {
  if (split_groups(sp.heads * sp.ng))
    launch_any<0, true>(g, sp, sp.ng, K, packed, use_fft, st, 0, Protect2Args{}, VEncArgs{});
  else
    launch_any<0, false>(g, sp, (sp.ng + K_GPB - 1) / K_GPB, K, packed, use_fft, st, 0, Protect2Args{}, VEncArgs{});
}

// false: too many heads for one grid, nothing done
bool launch_k_encode_protect2(const Geom& g, const void* K, uint8_t* packed_K, const void* V, uint8_t* packed_V,
                              hipStream_t st) {
  const Protect2Args p2 = protect2_args(g, V, packed_V);
  const EncodeSpan sp{g.T, g.ng, 0, g.nheads, 0};
  const long long gx = (g.ng + K_GPB - 1) / K_GPB, rows = ((p2.total + 3) / 4 + gx - 1) / gx;
  if (g.nheads + rows > 65535) return false;
  launch_any<1, false>(g, sp, (int)gx, K, packed_K, g.use_fft, st, (int)rows, p2, VEncArgs{});
  return true;
}

// Key and value coding passes of a residual block, MASK and RANK of its groups: one launch, one group per workgroup
// or, from split_groups() on, per wave.  (As three, 5.6 + 4.0 + 1.3 us and their gaps at 4 heads x 128 tokens, 28 layers took
// 446 us; as one of 5.8, 269; shared out, 3.5, and with the calls marshalled natively 115 to 132 on different hosts, whose time it is.)
bool launch_flush_encode(const Geom& g, const EncodeSpan& sp, float gamma, const void* K, const void* V,
                         uint8_t* packed_K, uint8_t* packed_V, hipStream_t st) {
  if (2 * sp.heads > 65535) return false;
  VEncArgs ve = v_encode_args(g, sp, 0, gamma, V, packed_V);
  ve.gpb = K_GPB;                                    // one grid for both
  if (g.n_s > 0) ve.mark_rank = g.n_s;
  if (split_groups(2 * sp.heads * sp.ng))
    launch_any<2, true>(g, sp, sp.ng, K, packed_K, g.use_fft, st, (int)sp.heads, Protect2Args{}, ve);
  else
    launch_any<2, false>(g, sp, (sp.ng + K_GPB - 1) / K_GPB, K, packed_K, g.use_fft, st, (int)sp.heads, Protect2Args{}, ve);
  return true;
}

// A whole call with few groups in two launches: ranges and MASK, then both coding passes and 2-bit rows, whose
// workgroups count ranks and select channels for themselves.  What bounds such a call is launches and latencies one after
// another: of three launches and 17.3 us for one head x 1568 tokens, 10 % fp16 rows, the token selection by one workgroup
// took 9; so 10.9 (4.1 + 7.2 on their own).  2-bit rows 18.7 -> 11.2; 4 heads x 3136 tokens 21.1 -> 13.6, 4 x 6272 22.6 -> 19.2, nothing protected
// 17.3 -> 14.8; 1008 groups 21.3 -> 16.5.  Every workgroup's own selection costs more than it saves from about five groups a
// compute unit on (1372 groups: 22.5 against 22.7, without rows 19.2 against 21.5; 1568: 24.8 against 28.6).
// false: too many, or a selection that is not few_selection(); nothing done.
void launch_k_range_select(const Geom& g, const void* K, void* ws, const float* scores, const int32_t* idx,
                           uint8_t* packed_V, bool few, hipStream_t st);
bool few_selection(const Geom& g, bool scores, bool alone);

bool launch_few_groups(const Geom& g, float gamma, const void* K, const void* V, void* ws, const float* scores,
                       const int32_t* idx, uint8_t* packed_K, uint8_t* packed_V, hipStream_t st) {
  if (g.nheads * g.ng > 4LL * device_cu_count() || !few_selection(g, scores != nullptr, true)) return false;
  launch_k_range_select(g, K, ws, scores, idx, packed_V, true, st);
  const EncodeSpan all{g.T, g.ng, 0, g.nheads, 0};
  VEncArgs ve = v_encode_args(g, all, g.n_s, gamma, V, packed_V);
  ve.range_ws = reinterpret_cast<const _Float16*>(ws);
  ve.chunks = g.range_chunks;
  ve.idx = reinterpret_cast<int32_t*>(packed_V + g.v_idx);
  const bool rows2 = g.n_s > 0 && g.sal_bits == 2;
  const Protect2Args p2 = rows2 ? protect2_args(g, V, packed_V) : Protect2Args{};
  const long long more = rows2 ? ((p2.total + 3) / 4 + g.ng - 1) / g.ng : 0;
  launch_any<3, true>(g, all, g.ng, K, packed_K, g.use_fft, st, (int)g.nheads, p2, ve, (int)more);
  return true;
}

}  // namespace vidkv
