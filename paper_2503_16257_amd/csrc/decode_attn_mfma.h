// MFMA decode attention over the packed cache (Eq. 3; Alg. 1, Decoding).
//
// One wave walks PAIRS of 32-token groups; the 16 "columns" of the score tiles
// are (group parity, query head <= 8).  All contractions run on
// v_mfma_f32_16x16x32_f16 with operands that are exact in fp16 and fp32
// accumulation:
//   * normal key channels (Eq. 5): rows = DFT coefficient slot, K = channels,
//     operand value -(+-s) = sign pattern | stored fp16 scale; columns carry
//     -q/16.  The result tile is already laid out as the B operand of the next
//     product,
//   * a 32-point inverse real DFT as a product with a constant matrix (split
//     into fp16 hi + lo parts, as is Y) giving scores[token][column],
//   * anomalous key channels (Eq. 4): code*s + z = (z + 1.5 s) + s0 (s/2) + s1 s
//     with s0, s1 = +-1 taken from the two code bits, rows = tokens, s as it is stored
//     against -q and -2 q; the column operand is masked by parity so both groups add
//     into the same score tile,
//   * P V: rows = columns of the score tile (probabilities are reused in place
//     as the A operand), K = tokens, columns = channels with operand +-1 / 0 from
//     the trits; the per-channel scale of Eq. 6 multiplies the fp32 result.
//
// Expanding one stored bit (or trit) into an fp16 operand element is what this
// kernel spends its time on, and two units can do it: the vector ALU (shift +
// mask pairs; a 64-bit shift serves two registers at once) and LDS (a byte of
// four trits indexes a 256-entry table of four fp16 values: one 8-byte read and
// nothing else).  Either alone saturates - LDS is shared by the four SIMDs of a
// compute unit - so the work is split: the key operands, which also carry their
// scale, are expanded on the ALU, the value operands through the table.
//
// Key and value records - and protected fp16 rows, four per instruction - go
// from memory straight into a per-wave LDS ring, one pair ahead
// (global_load_lds_dwordx4; lane l of a wave-wide transfer lands at M0 + 16 l,
// i.e. a record keeps its byte order; the two records of a pair are neighbours
// in memory and in the ring, so one run of 1 KB transfers covers both).
//
// Two-stage software pipeline per wave: while the keys of pair p are scored,
// the values of the wave's previous pair are multiplied by the
// probabilities that the previous step left in registers, as one interleaved
// instruction stream; the ring holds two key stages and two value stages.
//
// What orders the hand-offs through LDS.  Every ring, row and probability
// buffer is private to one wave, so no barrier is involved after the set-up
// (whose two __syncthreads order the shared tables, q and the permutation).
//   * transfer -> read: the compiler is not told that the transfer
//     instructions write LDS.  Each step begins with a written-out
//     "s_waitcnt vmcnt(0)" carrying a memory clobber: every transfer the wave
//     has issued - they were all issued in the previous step - has landed, and
//     no LDS read of the step can be moved above it.
//   * read -> overwrite: a stage is refilled by transfers issued only after
//     the step that read it has consumed the data in registers (the loads'
//     results are used, so their lgkmcnt waits have passed), and the transfer
//     statements carry a memory clobber, so the compiler keeps program order.
//   * probabilities and rescale factors staged with ordinary LDS stores are
//     read back by the same wave through ordinary loads: the compiler sees
//     both and inserts the lgkmcnt waits itself; LDS executes a wave's
//     operations in order.
// M0 is written inside the transfer statement and named in its clobber list;
// the kernel has no other user of M0.
//
// Softmax is online in the exp2 domain with a lazily raised running maximum
// shared by the two parities of a head.
//
// Protected value rows are a product of their own, [heads] x [protected tokens] x
// [channels], in batches of 16 fp16 rows (or one record of 32 rows at 2 bits): a wave
// walks consecutive pairs, gathers its protected tokens' probabilities into a list
// and multiplies a batch when it is full, since a pair has only a few such tokens (3
// of 64 at 5 %, 13 at 20 %) and one multiplication costs the same for 1 row as for 16.
// fp16 rows are transposed by the LDS read itself (ds_read_b64_tr_b16); a 2-bit code
// becomes an fp16 number where it stands (masked, then times 2^15: as the denormal number
// that its bits are, the products came out with fewer bits).  The probabilities enter as
// hi + lo halves, at no cost: 8 of the 16 operand rows would be empty.  (Rows one or two
// at a time on the vector ALU, 2-bit rows beyond the eighth of a pair straight from
// memory, and masks loaded with vector loads whose waits drained the transfers: 67.4 us
// against 13.9 for 28 query heads x 6272 tokens, n_a = 64, 20 % at 2 bits; 180 against 152
// for 64 sequences x 25088 tokens, n_a = 16, 5 % in fp16; 29.8 against 27.7 for one of 196000.)
#pragma once
#include <cstddef>
#include <type_traits>

#include "decode_attn.h"

namespace vidkv {

typedef unsigned short us2 __attribute__((ext_vector_type(2)));
typedef __attribute__((address_space(4))) uint32_t cu32;   // read with scalar loads

__device__ __forceinline__ float from_xor8(float v) {        // v(lane ^ 8): within a row of 16, 8 lanes on
  return __uint_as_float((uint32_t)__builtin_amdgcn_update_dpp(0, (int)__float_as_uint(v), 0x128, 0xF, 0xF, true));
}
// two floats -> packed fp16 pair, round to nearest even
__device__ __forceinline__ uint32_t pk_rne(float a, float b) {
  return h2_bits(__builtin_convertvector(f2{a, b}, h2));
}
__device__ __forceinline__ uint32_t pkrtz(float a, float b) {
  return __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_pkrtz(a, b));
}

// v << K as one 64-bit vector shift.  The empty asm makes all 64 result bits count as used,
// so the compiler cannot split the shift into two 32-bit ones.  (The shift itself must not
// be written as inline asm: the compiler does not insert the wait states that a vector
// write needs behind an MFMA still reading the same register when the write sits in an asm
// statement, and results came out wrong.)
template <int K>
__device__ __forceinline__ uint64_t shl64(uint64_t v) {
  uint64_t r = v << K;
  asm("" : "+v"(r));
  return r;
}
// byte B of w, times 8 (one instruction with a sub-dword source select; `three` is a 3 that the compiler does
// not see, which for byte 0 it would turn into a shift and a mask)
template <int B>
__device__ __forceinline__ uint32_t byte_x8(uint32_t w, uint32_t three) {
  return ((w >> (8 * B)) & 0xFFu) << three;
}

// Inverse-DFT operands.  split: 32 * (inverse real DFT matrix) as fp16 hi + lo parts, [2 lo + mt][lane][8 halves]: row
// t = 16 mt + x, k-slot (kb, i): i < 4 -> Re X[4kb+i], i >= 4 -> Im X[4kb+i-4] (Re X[16] when that index is 0).
// full: twice the matrix in fp32, [2 half + mt][lane][4]: k-slots i of the Re half (0) or the Im half (1).
// (Loaded: computed by every workgroup they took longer, 0.84 us, than q takes to arrive, where only one workgroup
// runs on a compute unit, and 250 vector instructions a wave beside others.)
struct IdftTab { uint32_t split[4][64][4]; float full[4][64][4]; };

constexpr IdftTab make_idft_tab() {
  IdftTab tab{};
  for (int n = 0; n < 4; ++n)
    for (int lane = 0; lane < 64; ++lane) {
      const int kb = lane >> 4, t = 16 * (n & 1) + (lane & 15);
      float w[8] = {};
      for (int i = 0; i < 8; ++i) {
        const int k = 4 * kb + (i & 3);
        w[i] = i < 4 ? (k == 0 ? 0.5f : cos32(k * t)) : k == 0 ? ((t & 1) ? -0.5f : 0.5f) : -cos32(k * t + 24);
        const _Float16 hi = (_Float16)(2.0f * w[i]);
        const _Float16 v = (n >> 1) ? (_Float16)(2.0f * w[i] - (float)hi) : hi;
        tab.split[n][lane][i >> 1] |= (uint32_t)__builtin_bit_cast(uint16_t, v) << (16 * (i & 1));
      }
      for (int i = 0; i < 4; ++i) tab.full[n][lane][i] = w[4 * (n >> 1) + i] * 0.125f;
    }
  return tab;
}

static __device__ const __align__(256) IdftTab kIdftTab = make_idft_tab();

// SAL: 0 no protected tokens, 1 protected rows in fp16, 2 protected rows as 2-bit records.
// FFT: normal key channels coded by Eq. 5 (true) or by Eq. 4 at 1 bit on the tokens (false);
// in the latter case slot = token and code * s + z = (z + s/2) + sigma * s/2, sigma = +-1,
// so the same sign-type operand serves, without the inverse DFT and with a constant term.
// FULL: the counts that a kernel in 32-bit arithmetic served before this one keep its accuracy:
//   * probabilities enter P V as three bf16 parts that add up to the fp32 number, whatever its size
//     (fp16 hi + lo parts are 0 below 2^-25 of the running maximum, where the softmax denominator
//     still counts the token: 196000 tokens at 2^-25.1 of one other lost 0.5 % of the output);
//   * protected rows' probabilities as hi + 2^-18 lo, two fp16 numbers (how many bits: at batch());
//   * the normal channels' q enters as it is, where the others' inverse DFT takes q/16 (half of it for a head with an
//     anomalous channel's element of 2^15 or more);
//   * the inverse DFT runs on v_mfma_f32_16x16x4_f32, on the fp32 sums and an fp32 matrix.
// The other counts have always had fp16 probabilities and -q/16.  What it costs is 48 instead of 32 products
// of a pair's values (the three parts are used as they are, in all rows: with the operand rows masked by parity, and
// the second part in the rows that the mask leaves, a third fewer products took more registers than there are) and
// 256 instead of 96 matrix-pipe cycles of its inverse DFT: n_a = 96, nothing protected, one layer of 196000 tokens
// 30.7 -> 33.7 us, 4 x 8 x 12544 tokens 86.6 -> 94.4, 2 x 3136 tokens 11.7 -> 11.5 (the 32-bit kernel: 309, 684, 24.2; by bit
// plane, since: 31.8, 79.8 and 8.8 with 100 residual tokens).
// (The DFT's products between the anomalous items instead of behind them: 34.0, 95.1.)
// TAIL: workgroups with split >= nsplit of the grid take residual tokens.  A variant of its own,
// since the branch costs the others 3 % (28 x 8 x 12544 tokens, n_a = 64: 597 us a step against 577).
template <int NA8, int SAL, bool FFT, bool TAIL>
__global__ __launch_bounds__(256, 2) void attn_mfma_kernel(AttnArgs a) {
  constexpr int NA = 8 * NA8, NN = D - NA;
  constexpr int NB = NN / 8;                 // normal 8-channel blocks
  constexpr int U = (NB + 3) / 4;            // K-steps over normal channels
  constexpr int NQ = NA / 4;                 // anomalous 4-channel quads
  constexpr int UA = (NQ + 3) / 4;           // K-steps over anomalous channels
  constexpr bool FULL = !(NA8 == 0 || NA8 == 1 || NA8 == 2 || NA8 == 4 || NA8 == 8 || NA8 == 16);
  constexpr bool IDFT = FFT && U > 0;        // scores of normal channels come through the inverse DFT
  constexpr int KREC = 12 * NA + 8 * NN;
  constexpr int OFF_AS = 8 * NA, OFF_AZ = 10 * NA, OFF_BITS = 12 * NA, OFF_META = 12 * NA + 4 * NN;
  constexpr int RING = 4 * KREC + 4 * VREC;  // a wave's ring: two stages of a pair's key records, two of its value records
  constexpr int BS = (SAL == 2) ? 32 : 16;   // protected rows multiplied at a time: a 2-bit record, or 16 fp16 rows
  constexpr int LCAP = 96;                   // a wave's list of protected probabilities: 32 waiting + a pair's 64
  constexpr int ROWB = (SAL == 2) ? PREC : BS * 2 * D;

  // Every argument that the way to the first requests needs, asked for at once: left to itself the compiler
  // loads each where it is used and waits for it, a cache miss per 64 bytes of arguments one after another
  // (from a wave's start to its last request 1.9 us, 0.9 so: 4 heads x 6272 tokens, n_a = 64, 2-bit rows).
  asm volatile("" :: "s"(a.q), "s"(a.kperm), "s"(a.krec), "s"(a.vrec), "s"(a.layer), "s"(a.B), "s"(a.H), "s"(a.Hq),
               "s"(a.rep), "s"(a.ng), "s"(a.ngc), "s"(a.gps), "s"(a.nsplit), "s"(a.early));
  if (SAL != 0) asm volatile("" :: "s"(a.vmask), "s"(a.vrank), "s"(a.vrows), "s"(a.n_s), "s"(a.npg));
  const int split = blockIdx.x, kvh = blockIdx.y, b = blockIdx.z;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);      // wave-uniform
  const int x16 = lane & 15, kb = lane >> 4;
  const int hcol = x16 & 7, par = x16 >> 3;          // column role: (parity, head)
  const int R = a.rep;
  const long long hd = ((long long)a.layer * a.B + b) * a.H + kvh;
  const f4 zero = f4{0.f, 0.f, 0.f, 0.f};

  // q and the channel permutation are needed only until the constant operands are built;
  // the lists of the protected tokens' probabilities take their place afterwards
  constexpr int PL_BYTES = (SAL != 0) ? 4 * LCAP * 8 * 4 : 0;
  constexpr int PRE_BYTES = 8 * D * 2 + D;
  // The table comes first: an LDS read reaches 64 KB beyond its address register, and where the table lay
  // behind that each of the 32 lookups of a pair took one more addition (n_a = 16, fp16 rows: 8 % of its vector
  // instructions).
  struct Lds {
    uint2 t_trit[256];             // byte -> 4 fp16 (FULL: bf16) numbers, number i = +1 / -1 / 0 from bits 2i (nonzero), 2i+1 (negative)
    u32x4 w_tab[4][64];            // per lane: inverse-DFT operands Wh[0], Wh[1], Wl[0], Wl[1] (FULL: fp32, [0] the Re half, [2] the Im half, of the first 16 tokens)
    float al16[4][16];             // per wave: rescale factors per column
    float mw[8][4], lw[8][4];      // [head][wave]
    alignas(256) uint8_t rowbuf[(SAL != 0) ? 4 : 1][(SAL != 0) ? ROWB : 16];   // per wave: the rows of the next batch
    alignas(256) uint8_t ring[4][RING];  // per wave: 2 key stages, 2 value stages; reused for the wave's partial output
    alignas(16) uint8_t pre_s[PRE_BYTES > PL_BYTES ? PRE_BYTES : PL_BYTES];
  };
  __shared__ __align__(256) Lds lds;
  auto& t_trit = lds.t_trit;
  auto& w_tab = lds.w_tab;
  auto& al16 = lds.al16;
  auto& mw = lds.mw;
  auto& lw = lds.lw;
  auto& rowbuf = lds.rowbuf;
  auto& ring = lds.ring;
  auto& pre_s = lds.pre_s;
  _Float16 (*qs)[D] = reinterpret_cast<_Float16 (*)[D]>(pre_s);
  uint8_t* perm_s = pre_s + 8 * D * 2;
  float (*plist)[LCAP][8] = reinterpret_cast<float (*)[LCAP][8]>(pre_s);   // per wave, a ring: probabilities [protected token][head]
  static_assert(sizeof(float) * 8 * D <= RING, "a wave's partial output must fit its ring");

  if (TAIL && split >= a.nsplit) {
    // (arguments read anew here, so that the main path's registers do not hold them)
    const __attribute__((address_space(4))) AttnArgs* ap =
        (const __attribute__((address_space(4))) AttnArgs*)__builtin_amdgcn_kernarg_segment_ptr();
    asm volatile("" : "+s"(ap));
    static_assert(sizeof(TailLds) <= sizeof(lds.ring), "the residual part must fit the rings");
    attn_tail_part(*(const AttnArgs*)ap, split - ap->nsplit, kvh, b, *reinterpret_cast<TailLds*>(&ring[0][0]));
    return;
  }

  // ---------------- transfers
  const int npairs = (a.ng + 1) >> 1;
  // the waves take turns at the split's pairs - or, when there are protected rows, each walks a
  // contiguous run of them, so that its rows are consecutive in ROWS
  constexpr int PSTEP = (SAL != 0) ? 1 : 4;
  const int s_begin = split * a.gps;
  const int s_end = min(npairs, s_begin + a.gps), s_n = max(0, s_end - s_begin);
  const int p_begin = (SAL != 0) ? s_begin + (s_n * wave) / 4 : s_begin + wave;
  const int p_end = (SAL != 0) ? s_begin + (s_n * (wave + 1)) / 4 : s_end;

  const uint8_t* krec_base = a.krec + hd * a.ngc * (long long)KREC;
  const uint8_t* vrec_base = a.vrec + hd * a.ngc * (long long)VREC;

  // M0 is the LDS base of a transfer.  It is written inside the asm statement and named in
  // its clobber list; this kernel has no other user of M0 (no indirect register indexing,
  // no compiler-generated LDS transfers).
  auto dma16 = [&](const uint8_t* g, uint32_t lds_byte) {
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off nt"
                 :: "s"(lds_byte), "v"(g) : "memory", "m0");
  };
  // ring of a wave: key stages 0, 1, then value stages 0, 1 (a stage = the two groups of a pair)
  const uint32_t ring_lds = (uint32_t)reinterpret_cast<uintptr_t>(&ring[0][0]) + (uint32_t)(wave * RING);
  const uint8_t* ring_w = &ring[wave][0];
  // The two records of a pair are neighbours in memory and in the stage: one run of 1 KB
  // instructions covers both, the last one the last 1 KB (it brings some bytes twice, and no lane is
  // masked).  The instruction's offset counts for both sides.  (A last pair with one group fetches that
  // group twice, so that the unused half of the stage holds finite numbers.)
  constexpr int NDMA_K = (2 * KREC + 1023) / 1024;       // fewest instructions of one key transfer
  constexpr int NDMA_V = (2 * VREC + 1023) / 1024;
  const uint32_t lane16 = lane * 16;
  // (M0 is written for every transfer; where it already holds the value, no wait state is needed in between.
  // The first transfer of a statement stands five wait states behind its beginning: the compiler does not see
  // that it reads SRC, which a vector instruction may have written.)
#define VIDKV_DMA(DST, AT, SRC, OFF) "s_mov_b32 m0, " DST "\n\ts_nop 1\n\tglobal_load_lds_dwordx4 " AT ", " SRC " offset:" OFF " nt\n\t"
#define VIDKV_DMA_MORE(DST, AT, SRC, OFF) "s_mov_b32 m0, " DST "\n\tglobal_load_lds_dwordx4 " AT ", " SRC " offset:" OFF " nt\n\t"
  auto fetch_run = [&](const uint8_t* src, uint32_t dst, auto nbytes_c) {
    constexpr int NBYTES = decltype(nbytes_c)::value;
    const uint32_t at = lane16;
    asm volatile("s_nop 1\n\t" VIDKV_DMA("%0", "%1", "%2", "0")
                 ".if %4 > 2048\n\t" VIDKV_DMA_MORE("%0", "%1", "%2", "1024") ".endif\n\t"
                 VIDKV_DMA_MORE("%0", "%1", "%2", "%3")
                 :: "s"(dst), "v"(at), "s"(src), "n"(NBYTES - 1024), "n"(NBYTES) : "memory", "m0");
  };
  // the pair pp of a head's records into the stage at dst, if `go`; the branches are inside the statement,
  // so that what surrounds it stays one piece of straight code
  auto fetch_pair = [&](const uint8_t* base, auto rec_c, int pp, uint32_t dst, bool go) {
    constexpr int REC = decltype(rec_c)::value;
    const uint32_t at = lane16;
    const int g = 2 * pp + 1 < a.ng ? 2 * pp : a.ng - 1;
    const int what = go ? (2 * pp + 1 < a.ng ? 1 : 2) : 0;
    const uint8_t* src = base + (long long)g * REC;
    asm volatile("s_cmp_eq_u32 %0, 1\n\ts_cbranch_scc0 .Lone%=\n\t"
                 VIDKV_DMA("%1", "%3", "%4", "0")
                 ".if %8 > 2048\n\t" VIDKV_DMA_MORE("%1", "%3", "%4", "1024") ".endif\n\t"
                 VIDKV_DMA_MORE("%1", "%3", "%4", "%5")
                 "s_branch .Lend%=\n"
                 ".Lone%=:\n\t"
                 "s_cmp_eq_u32 %0, 0\n\ts_cbranch_scc1 .Lend%=\n\t"
                 VIDKV_DMA("%1", "%3", "%4", "0")
                 ".if %7 > 1024\n\t" VIDKV_DMA_MORE("%1", "%3", "%4", "%6") ".endif\n\t"
                 VIDKV_DMA("%2", "%3", "%4", "0")
                 ".if %7 > 1024\n\t" VIDKV_DMA_MORE("%2", "%3", "%4", "%6") ".endif\n"
                 ".Lend%=:"
                 :: "s"(what), "s"(dst), "s"(dst + REC), "v"(at), "s"(src), "n"(2 * REC - 1024), "n"(REC - 1024),
                    "n"(REC), "n"(2 * REC) : "memory", "m0", "scc");
  };
  auto fetch_keys = [&](int pp, int st, bool go) {
    fetch_pair(krec_base, std::integral_constant<int, KREC>{}, pp, ring_lds + st * 2 * KREC, go);
  };
  auto fetch_values = [&](int pp, int st, bool go) {
    fetch_pair(vrec_base, std::integral_constant<int, VREC>{}, pp, ring_lds + 4 * KREC + st * 2 * VREC, go);
  };
  // Protected tokens.  The probabilities of a wave's protected tokens are gathered, in token
  // order, into a list in LDS; whenever it holds a batch (BS of them) their rows - consecutive in
  // ROWS, requested when the batch before was done - are multiplied on the matrix cores.  Masks:
  // of the pair whose probabilities are collected next (v), the pair being scored (c), the next (n).
  uint32_t sm0v = 0, sm1v = 0, sm0c = 0, sm1c = 0, sm0n = 0, sm1n = 0;
  auto load_masks = [&](int pp, uint32_t& s0, uint32_t& s1) {
    s0 = s1 = 0;
    if (SAL != 0) {
      // scalar loads (constant address space, no branch): as vector loads the compiler waited
      // for each of them, and with it for every transfer in flight, at the end of every step
      const cu32* mk = (const cu32*)a.vmask + (size_t)b * a.ngc;
      const uint32_t m0 = mk[min(2 * pp, a.ng - 1)], m1 = mk[min(2 * pp + 1, a.ng - 1)];
      s0 = pp < p_end ? m0 : 0u;
      s1 = pp < p_end && 2 * pp + 1 < a.ng ? m1 : 0u;
    }
  };
  int rb = 0, rk_end = 0;                    // rank of the first row of the batch being filled; end of the wave's rows
  int lpos = 0, lcnt = 0, lfirst = 0;        // where that batch starts in the ring, entries in it and behind it, first valid entry
  const uint32_t rowbuf_lds = (uint32_t)reinterpret_cast<uintptr_t>(&rowbuf[(SAL != 0) ? wave : 0][0]);
  auto fetch_rows = [&]() {
    if (SAL == 1) {
      // four rows (1 KB) per instruction; row r keeps its 16-byte pieces in the order
      // piece ^ 2 (r & 7), so that the transposing reads of a batch spread over the banks.
      const uint8_t* base = reinterpret_cast<const uint8_t*>(a.vrows + (hd * a.n_s + rb) * D);
      uint32_t ln = lane;
      asm volatile("" : "+v"(ln));
      const int r0 = ln >> 4;
      if (rb + BS <= a.n_s) {
        // a whole batch of the head's rows is there (those past the wave's end are not used): rows 4 j + r0, and
        // piece ^ 2 (r & 7) differs by 8 pieces between even and odd j
        const uint32_t at = r0 * (2 * D) + ((ln & 15) ^ (2 * r0)) * 16, at1 = at ^ 128;
        asm volatile("s_cmp_lt_i32 %0, %1\n\ts_cbranch_scc0 .Lend%=\n\t"
                     VIDKV_DMA("%2", "%3", "%5", "0")
                     VIDKV_DMA_MORE("%2", "%4", "%5", "1024")
                     VIDKV_DMA_MORE("%2", "%3", "%5", "2048")
                     VIDKV_DMA_MORE("%2", "%4", "%5", "3072")
                     ".Lend%=:"
                     :: "s"(rb), "s"(rk_end), "s"(rowbuf_lds), "v"(at), "v"(at1), "s"(base) : "memory", "m0", "scc");
      } else {
        const int n = min(BS, rk_end - rb);
#pragma unroll
        for (int j = 0; j < BS / 4; ++j) {
          const int r = 4 * j + r0, x16 = ln & 15;
          if (4 * j < n && r < n) dma16(base + r * 2 * D + (x16 ^ (2 * (r & 7))) * 16, rowbuf_lds + j * 1024u);
        }
      }
    } else if (rb < rk_end) {
      fetch_run(reinterpret_cast<const uint8_t*>(a.vrows) + (hd * a.npg + (rb >> 5)) * (long long)PREC, rowbuf_lds,
                std::integral_constant<int, PREC>{});
    }
  };
  int p = p_begin;

  // What the wave has to know of its protected tokens, asked for in front of the transfers and looked at behind
  // the first barrier (behind the transfers, with a wait at once, it held up the rows' request by 0.4 us)
  uint32_t rank0 = 0, rank1 = 0, mask1 = 0, mk0 = 0, mk1 = 0, mk2 = 0, mk3 = 0;
  if (SAL != 0) {
    const cu32* rk = (const cu32*)a.vrank + (size_t)b * a.ngc;
    const cu32* mk = (const cu32*)a.vmask + (size_t)b * a.ngc;
    const int last = a.ng - 1, g0 = 2 * p_begin, g1 = max(0, min(2 * p_end - 1, last));
    rank0 = rk[min(g0, last)]; rank1 = rk[g1]; mask1 = mk[g1];
    mk0 = mk[min(g0, last)]; mk1 = mk[min(g0 + 1, last)];
    mk2 = mk[min(g0 + 2, last)]; mk3 = mk[min(g0 + 3, last)];
    __builtin_amdgcn_sched_barrier(0);
  }

  // ---------------- set-up: the inverse-DFT operands (1 KB each wave, where there are any), q and the channel
  // permutation (wave 0 asks for them) go straight to LDS, the first pair's key records are requested right behind
  // them, and only the former are waited for: the operands are built while the records are on their way
  if (IDFT) {
    const uint32_t at = lane16;
    asm volatile("s_nop 1\n\t" VIDKV_DMA("%0", "%1", "%2", "0")
                 :: "s"((uint32_t)reinterpret_cast<uintptr_t>(&w_tab[0][0]) + 1024u * wave), "v"(at),
                    "s"(reinterpret_cast<const uint8_t*>(&kIdftTab) + (FULL ? offsetof(IdftTab, full) : 0) + 1024 * wave) : "memory", "m0");
  }
  if (wave == 0) {
    const uint8_t* qsrc = reinterpret_cast<const uint8_t*>(a.q + ((long long)b * a.Hq + kvh * R) * D);
    const uint32_t q_lds = (uint32_t)reinterpret_cast<uintptr_t>(pre_s);
    const int qbytes = R * D * 2;
    // head r keeps its 16-byte pieces in the order piece ^ 2 r: one channel of the 8 heads, read by the 16
    // columns of a wave at a time, lies in 8 different groups of banks (in the same one: the operands of
    // q took 0.95 us, 1.4 with eight waves on a compute unit; now 0.5 and 0.75)
    const int q_off = (lane * 16) ^ ((lane >> 4) * 32);
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off"
                 :: "s"(q_lds), "v"(qsrc + (lane * 16 < qbytes ? q_off : 0)) : "memory", "m0");
    if (1024 + lane * 16 < qbytes)
      asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off"
                   :: "s"(q_lds + 1024u), "v"(qsrc + 1024 + (q_off ^ 128)) : "memory", "m0");
    if (lane < D / 16)
      asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off"
                   :: "s"(q_lds + 8u * D * 2u), "v"(a.kperm + hd * D + lane * 16) : "memory", "m0");
  }
  fetch_keys(p, 0, p < p_end);
  fetch_values(p, 0, p < p_end && a.early);
  // ---------------- the expansion table of the value operands (behind the first requests, whose latency it fills)
  {
    uint32_t h[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const uint32_t f = ((uint32_t)tid >> (2 * i)) & 3u;
      h[i] = (f & 1u) ? ((f & 2u) ? 0x8000u : 0u) | (FULL ? 0x3F80u : 0x3C00u) : 0u;
    }
    t_trit[tid] = uint2{h[0] | (h[1] << 16), h[2] | (h[3] << 16)};
  }

  // the inverse-DFT operands, q and the permutation have landed: at least this many transfers were asked for later
  if (p < p_end && a.early) asm volatile("s_waitcnt vmcnt(%0)" :: "n"(NDMA_K + NDMA_V) : "memory");
  else if (p < p_end) asm volatile("s_waitcnt vmcnt(%0)" :: "n"(NDMA_K) : "memory");
  else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __syncthreads();
  if (SAL != 0) {
    if (p_begin < p_end) {
      rb = (int)rank0;
      rk_end = (int)rank1 + __popc(mask1);
      if (SAL == 2) {                        // batches are whole records
        lfirst = lcnt = rb & 31;
        rb &= ~31;
      }
      sm0c = mk0;
      sm1c = 2 * p + 1 < a.ng ? mk1 : 0u;
    }
    if (p_begin + 1 < p_end) {
      sm0n = mk2;
      sm1n = 2 * p + 3 < a.ng ? mk3 : 0u;
    }
  }
  const bool hv = hcol < R;
  const _Float16* qrow = &qs[hv ? hcol : 0][0];
  const uint32_t qswz = hv ? hcol * 0x10101010u : 0u;        // (four channels' numbers at a time)
  // The permutation bytes of my channel blocks and quads come in one LDS read each, then
  // every q element in one batch of independent reads (no branch around a read: absent
  // blocks read a valid block and are zeroed afterwards).
  Op Bn[2][U > 0 ? U : 1];                   // normal channels: -q h (FFT but FULL: -q h / 16; -q/2 with no others) at channels 8 (4u+kb) + e, only in my parity
  Op Ba[2][UA > 0 ? UA : 1];                 // anomalous: -q h of a quad's 4 channels, then -2 q h, only in my parity
  float sc2 = a.scale2;                      // sum -> score in the exp2 domain (the sums are 2 h times the scores')
  {
    uint2 pb[U > 0 ? U : 1];
    uint32_t pq[UA > 0 ? UA : 1];
#pragma unroll
    for (int u = 0; u < U; ++u)
    {
      pb[u] = *reinterpret_cast<const uint2*>(&perm_s[NA + 8 * min(4 * u + kb, NB - 1)]);
      pb[u].x ^= qswz;
      pb[u].y ^= qswz;
    }
#pragma unroll
    for (int ua = 0; ua < UA; ++ua)
      pq[ua] = *reinterpret_cast<const uint32_t*>(&perm_s[4 * min(4 * ua + kb, NQ - 1)]) ^ qswz;
    _Float16 qn[U > 0 ? U : 1][8], qa[UA > 0 ? UA : 1][4];
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
      for (int e = 0; e < 8; ++e) qn[u][e] = qrow[((e < 4 ? pb[u].x : pb[u].y) >> (8 * (e & 3))) & 0xFFu];
#pragma unroll
    for (int ua = 0; ua < UA; ++ua)
#pragma unroll
      for (int r = 0; r < 4; ++r) qa[ua][r] = qrow[(pq[ua] >> (8 * r)) & 0xFFu];
    // The second bit's operand is 2 q h: h = 1, or 1/2 for a head with an anomalous channel's element whose double is no fp16
    // number.  (Halves for the first bit instead lose the last bit of an element below 2^-13: 128 keys of 60000 against q = 15 2^-24
    // gave scores 7 % off.)  Without anomalous channels and inverse DFT the sums are the scores themselves.
    constexpr bool TWICE = UA > 0 || FFT;
    if (TWICE) sc2 *= 0.5f;
    const _Float16 cn = (_Float16)(FFT && !FULL ? -0.0625f : TWICE ? -1.0f : -0.5f);
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const bool ok = hv && (4 * u + kb) < NB;
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const _Float16 v = ok ? (_Float16)(qn[u][e] * cn) : (_Float16)0.0f;
        Bn[0][u].v[e] = par ? (_Float16)0.0f : v;
        Bn[1][u].v[e] = par ? v : (_Float16)0.0f;
      }
    }
    us2 most = {0, 0};                       // of the magnitudes of 2 q, as bit patterns
    auto anomalous_operands = [&](_Float16 h) {
#pragma unroll
      for (int ua = 0; ua < UA; ++ua) {
        const bool ok = hv && (4 * ua + kb) < NQ;
#pragma unroll
        for (int plane = 0; plane < 2; ++plane)
#pragma unroll
          for (int r = 0; r < 4; r += 2) {
            h2 x = h2{qa[ua][r], qa[ua][r + 1]} * h2{h, h};
            if (plane) x += x;
            const uint32_t w = ok ? h2_bits(x) : 0u;
            if (plane) most = __builtin_elementwise_max(most, __builtin_bit_cast(us2, w & 0x7FFF7FFFu));
            Ba[0][ua].u[2 * plane + r / 2] = par ? 0u : w;
            Ba[1][ua].u[2 * plane + r / 2] = par ? w : 0u;
          }
      }
    };
    anomalous_operands((_Float16)-1.0f);
    if (UA > 0) {
      const bool inf = most[0] >= 0x7C00 || most[1] >= 0x7C00;
      if (__builtin_expect(__any(inf), 0)) {                      // (as a maximum in front of the operands it was 1 % of a step: 28 layers x 6272 tokens 294.3 us, 289.0 so)
        const bool big = swap_max16(swap_max32(inf ? 1.0f : 0.0f)) > 0.0f;
        anomalous_operands((_Float16)(big ? -0.5f : -1.0f));
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
          for (int grp = 0; grp < 2; ++grp)
#pragma unroll
            for (int e = 0; e < 8; ++e) Bn[grp][u].v[e] *= (_Float16)(big ? 0.5f : 1.0f);
        if (big) sc2 *= 2.0f;
      }
    }
  }
  __syncthreads();                           // every wave is done with q and the permutation
  const uint32_t keep0 = par ? 0u : ~0u, keep1 = ~keep0;    // which group's P V product my column feeds
  const uint8_t* ttrit_b = reinterpret_cast<const uint8_t*>(&t_trit[0]);
  uint32_t three = 3;
  asm("" : "+v"(three));

  // ---------------- running state
  // o[m][i]: row 4kb+i = (parity, head) column of the score tile, channel 16 m + x16;
  // holds sum p * code * s of the quantized tokens.  Protected tokens add to the same sums: the
  // high parts of their probabilities in the rows of parity 0, the low parts in those of parity 1.
  f4 o[8];
#pragma unroll
  for (int m = 0; m < 8; ++m) o[m] = zero;
  float m_run = -INFINITY, l_run = 0.0f;     // of my column (shared by both parities of a head)
  uint32_t pp[4] = {0u, 0u, 0u, 0u};         // probabilities of the pair whose values come next
  uint32_t pm[4] = {0u, 0u, 0u, 0u}, pl[4] = {0u, 0u, 0u, 0u};   // ... their second and third parts (FULL)

  // ---------------- the pieces of one step.  Stage numbers are compile-time constants (the
  // loop alternates two instances of the step) so that every LDS address of the records is a
  // register plus an immediate.

  // What a lane reads first of a step, in one batch ahead of everything else (and ahead of
  // the transfer requests of the step: LDS reads issued behind those were seen to wait for
  // them): every sign word and code byte that it expands, the anomalous channels' scale and
  // zero point, the value words and scales.
  constexpr bool HOP_SZ = UA <= 2;           // scale and zero point in the batch too (registers allow it)
  struct FirstHop {
    uint32_t wn[2][U > 0 ? U : 1], wi[2][U > 0 ? U : 1], wa[2][UA > 0 ? UA : 1][2];
    uint2 as[2][HOP_SZ && UA > 0 ? UA : 1], az[2][HOP_SZ && UA > 0 ? UA : 1];
    u32x4 vw[2], sv;
  };
  auto first_hop = [&](auto ks_c, auto dok_c, auto dov_c, FirstHop& hop) {
    constexpr int KS = decltype(ks_c)::value;
    constexpr bool DO_K = decltype(dok_c)::value, DO_V = decltype(dov_c)::value;
    const uint8_t* stage = ring_w + KS * 2 * KREC;
    const uint8_t* vst = ring_w + 4 * KREC + (KS ^ 1) * 2 * VREC;
    if (DO_K) {
#pragma unroll
      for (int grp = 0; grp < 2; ++grp) {
        const uint8_t* rec = stage + grp * KREC;
#pragma unroll
        for (int u = 0; u < U; ++u) {
          const uint8_t* wp = rec + OFF_BITS + (min(4 * u + kb, NB - 1) * 16 + x16) * 2;
          hop.wn[grp][u] = *reinterpret_cast<const uint16_t*>(wp);   // both tiles' bits (the upper 8 never reach a sign position)
          hop.wi[grp][u] = wp[1];                                     // the second tile's alone
        }
#pragma unroll
        for (int ua = 0; ua < UA; ++ua) {
          const int quad = min(4 * ua + kb, NQ - 1);
#pragma unroll
          for (int mt = 0; mt < 2; ++mt) hop.wa[grp][ua][mt] = rec[(16 * mt + x16) * NQ + quad];
          if (HOP_SZ) {
            hop.as[grp][ua] = *reinterpret_cast<const uint2*>(rec + OFF_AS + quad * 8);
            hop.az[grp][ua] = *reinterpret_cast<const uint2*>(rec + OFF_AZ + quad * 8);
          }
        }
      }
    }
    if (DO_V) {
      hop.vw[0] = *reinterpret_cast<const u32x4*>(vst + lane * 16);
      hop.vw[1] = *reinterpret_cast<const u32x4*>(vst + VREC + lane * 16);
      hop.sv = *reinterpret_cast<const u32x4*>(vst + (kb >> 1) * VREC + 1024 + x16 * 16);
    }
  };

  // Scores of one pair from its key records (DO_K; key stage KS) and P V of the pair before
  // it from its value records and the packed probabilities pp (DO_V; value stage KS ^ 1),
  // as ONE instruction stream: the work items of the two - a K-step of channels, a channel
  // tile of values - alternate, each with the LDS reads of its successor in front, and the
  // scheduler is kept from pulling the two chains apart again.  Leaves S[token tile][4]
  // (per column) and the additive constant of the anomalous (and non-FFT) part.
  auto scores_and_values = [&](auto ks_c, auto dok_c, auto dov_c, const FirstHop& hop, f4 (&S)[2], float& cst) {
    constexpr int KS = decltype(ks_c)::value;
    constexpr bool DO_K = decltype(dok_c)::value, DO_V = decltype(dov_c)::value;
    constexpr int NKA = DO_K ? 2 * UA : 0, NKN = DO_K ? 2 * U : 0, NK = NKA + NKN;
    const uint8_t* stage = ring_w + KS * 2 * KREC;
    const uint32_t (&wn)[2][U > 0 ? U : 1] = hop.wn;
    const uint32_t (&wi)[2][U > 0 ? U : 1] = hop.wi;
    const uint32_t (&wa)[2][UA > 0 ? UA : 1][2] = hop.wa;
    u32x4 vw[2];
    Op sv, Ap[2];                                // sv: Eq. 6 scales of channels 16 m + x16, my rows' group
    if (DO_V) {
      vw[0] = hop.vw[0];
      vw[1] = hop.vw[1];
      sv.q = hop.sv;
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        Ap[0].u[r] = pp[r] & keep0;
        Ap[1].u[r] = pp[r] & keep1;
      }
    }
    S[0] = zero; S[1] = zero;
    f4 accRe = zero, accIm = zero, accCn = zero, accCs = zero, accC[3] = {zero, zero, zero};   // my column's group only: the operands are masked

    // ---- the work items
    // scales of the normal K-step n = (group, u)
    auto load_meta = [&](int n, Op& sre, Op& sim) {
      const int grp = n / (U > 0 ? U : 1), u = n % (U > 0 ? U : 1);
      const uint8_t* rec = stage + grp * KREC;
      const int blk = min(4 * u + kb, NB - 1);
      sre.q = *reinterpret_cast<const u32x4*>(rec + OFF_META + (blk * 2) * 16);
      sim.q = *reinterpret_cast<const u32x4*>(rec + OFF_META + (blk * 2 + ((FFT && x16) ? 1 : 0)) * 16);
    };
    // normal channels: Y[slot][col] per group, K = channels
    auto normal_item = [&](int n, const Op& sre, const Op& sim) {
      const int grp = n / (U > 0 ? U : 1), u = n % (U > 0 ? U : 1);
      const uint32_t w = wn[grp][u], w2 = wi[grp][u];
      Op Are, Aim;
      // bit e of a byte: channel e.  In x | x << 15 a channel pair (2r, 2r+1) sits 15 - 2r
      // below bits (15, 31); with the first tile's word in the lower and the second tile's in
      // the upper half, one 64-bit shift positions both (what it carries into the upper word
      // stays below bit 15)
      const uint64_t x2 = ((uint64_t)(w2 | (w2 << 15)) << 32) | (w | (w << 15));
      const uint64_t s0 = shl64<15>(x2), s1 = shl64<13>(x2), s2 = shl64<11>(x2), s3 = shl64<9>(x2);
      Are.u[0] = ((uint32_t)s0 & 0x80008000u) | sre.u[0]; Aim.u[0] = ((uint32_t)(s0 >> 32) & 0x80008000u) | sim.u[0];
      Are.u[1] = ((uint32_t)s1 & 0x80008000u) | sre.u[1]; Aim.u[1] = ((uint32_t)(s1 >> 32) & 0x80008000u) | sim.u[1];
      Are.u[2] = ((uint32_t)s2 & 0x80008000u) | sre.u[2]; Aim.u[2] = ((uint32_t)(s2 >> 32) & 0x80008000u) | sim.u[2];
      Are.u[3] = ((uint32_t)s3 & 0x80008000u) | sre.u[3]; Aim.u[3] = ((uint32_t)(s3 >> 32) & 0x80008000u) | sim.u[3];
      accRe = mma(Are, Bn[grp][u], accRe);
      accIm = mma(Aim, Bn[grp][u], accIm);
      if (!FFT) {
        // constant term, rows all equal: z and s against the same operand, apart: the score takes 2 z + s
        const uint8_t* rec = stage + grp * KREC;
        const int blk = min(4 * u + kb, NB - 1);
        Op zq;
        zq.q = *reinterpret_cast<const u32x4*>(rec + OFF_META + (blk * 2 + 1) * 16);
        accCn = mma(zq, Bn[grp][u], accCn);
        accCs = mma(sre, Bn[grp][u], accCs);
      }
    };
    // anomalous channels: rows = tokens, K = (bit plane, channel); the column operand is
    // zero outside my parity, so both groups add into S directly
    // scale and zero point of the anomalous K-step n, read one item ahead (n_a = 64, 28 x 8 x 12544
    // tokens: 570 us a step with the reads in front of their use, 558 so)
    auto load_sz = [&](int n, uint2& as, uint2& az) {
      const int grp = n / (UA > 0 ? UA : 1), ua = n % (UA > 0 ? UA : 1);
      const uint8_t* rec = stage + grp * KREC;
      const int quad = min(4 * ua + kb, NQ - 1);
      as = *reinterpret_cast<const uint2*>(rec + OFF_AS + quad * 8);
      az = *reinterpret_cast<const uint2*>(rec + OFF_AZ + quad * 8);
    };
    auto anomalous_item = [&](int n, uint2 as, uint2 az) {
      const int grp = n / (UA > 0 ? UA : 1), ua = n % (UA > 0 ? UA : 1);
      const uint2 s4 = HOP_SZ ? hop.as[grp][ua] : as, z4 = HOP_SZ ? hop.az[grp][ua] : az;   // of the quad's 4 channels
      // Code bytes of my two tokens (tiles mt = 0, 1): bits (2r, 2r+1) of a byte are the code of channel r.  In
      // x | x << 14 one plane's bits of channels (0, 1) lie 16 apart, and (2, 3) likewise 4 further up; from
      // there as with the sign words.  By plane and not by channel, so that scales and zero points are operands as they
      // stand in the record: an instruction for each of (s/2, s) and (z, 0) before, 64 of a pair's 380 at n_a = 64.
      const uint32_t w0 = wa[grp][ua][0], w1 = wa[grp][ua][1];
      const uint64_t x2 = ((uint64_t)(w1 | (w1 << 14)) << 32) | (w0 | (w0 << 14));
      Op A0, A1;
      const uint64_t s0 = shl64<15>(x2), s1 = shl64<11>(x2), s2 = shl64<14>(x2), s3 = shl64<10>(x2);
      A0.u[0] = ((uint32_t)s0 & 0x80008000u) | s4.x; A1.u[0] = ((uint32_t)(s0 >> 32) & 0x80008000u) | s4.x;
      A0.u[1] = ((uint32_t)s1 & 0x80008000u) | s4.y; A1.u[1] = ((uint32_t)(s1 >> 32) & 0x80008000u) | s4.y;
      A0.u[2] = ((uint32_t)s2 & 0x80008000u) | s4.x; A1.u[2] = ((uint32_t)(s2 >> 32) & 0x80008000u) | s4.x;
      A0.u[3] = ((uint32_t)s3 & 0x80008000u) | s4.y; A1.u[3] = ((uint32_t)(s3 >> 32) & 0x80008000u) | s4.y;
      S[0] = mma(A0, Ba[grp][ua], S[0]);
      S[1] = mma(A1, Ba[grp][ua], S[1]);
      // the constant z + 1.5 s, 2 h times it: rows all equal, s against both planes' operands, z against the second's
      const h8 q8 = Ba[grp][ua].v;
      const h4 q1 = __builtin_shufflevector(q8, q8, 0, 1, 2, 3), q2 = __builtin_shufflevector(q8, q8, 4, 5, 6, 7);
      const h4 sv4 = __builtin_bit_cast(h4, s4), zv4 = __builtin_bit_cast(h4, z4);
      // (three sums, so that none waits for the product in front of it)
      accC[0] = __builtin_amdgcn_mfma_f32_16x16x16f16(sv4, q1, accC[0], 0, 0, 0);
      accC[1] = __builtin_amdgcn_mfma_f32_16x16x16f16(sv4, q2, accC[1], 0, 0, 0);
      accC[2] = __builtin_amdgcn_mfma_f32_16x16x16f16(zv4, q2, accC[2], 0, 0, 0);
    };
    // table entries of value tile m, both groups: byte (m & 1) of word m >> 1 holds the even
    // token slots 0, 2, 4, 6, byte 2 + (m & 1) the odd slots 1, 3, 5, 7
    auto lookup = [&](int m, uint2 (&E)[2], uint2 (&O)[2]) {
#pragma unroll
      for (int grp = 0; grp < 2; ++grp) {
        const uint32_t w = vw[grp][m >> 1];
        const uint32_t ae = (m & 1) ? byte_x8<1>(w, three) : byte_x8<0>(w, three);
        const uint32_t ao = (m & 1) ? byte_x8<3>(w, three) : byte_x8<2>(w, three);
        E[grp] = *reinterpret_cast<const uint2*>(ttrit_b + ae);
        O[grp] = *reinterpret_cast<const uint2*>(ttrit_b + ao);
      }
    };
    // P V of tile m: C[column][channel 16 m + x16] = sum_t p * code; o += s * C follows one tile later, when
    // the products are done (right behind them a wave waits 8 issue slots for each tile)
    auto value_tile = [&](int m, const uint2 (&E)[2], const uint2 (&O)[2]) -> f4 {
      f4 C = zero;
      if (FULL) {
        // every row times either group's values; my rows' parity says which of the two counts
        f4 Cg[2] = {zero, zero};
#pragma unroll
        for (int grp = 0; grp < 2; ++grp) {
          Op Bv, P3;
          Bv.u[0] = E[grp].x; Bv.u[1] = E[grp].y; Bv.u[2] = O[grp].x; Bv.u[3] = O[grp].y;
          P3.q = u32x4{pl[0], pl[1], pl[2], pl[3]};
          Cg[grp] = mma_bf16(P3, Bv, Cg[grp]);
          P3.q = u32x4{pm[0], pm[1], pm[2], pm[3]};
          Cg[grp] = mma_bf16(P3, Bv, Cg[grp]);
          P3.q = u32x4{pp[0], pp[1], pp[2], pp[3]};
          Cg[grp] = mma_bf16(P3, Bv, Cg[grp]);
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) C[i] = (kb >> 1) ? Cg[1][i] : Cg[0][i];
      } else {
#pragma unroll
        for (int grp = 0; grp < 2; ++grp) {
          Op Bv;
          Bv.u[0] = E[grp].x; Bv.u[1] = E[grp].y; Bv.u[2] = O[grp].x; Bv.u[3] = O[grp].y;
          C = mma(Ap[grp], Bv, C);
        }
      }
      return C;
    };
    auto add_tile = [&](int m, const f4& C) {
      const float sc = (float)sv.v[m];
#pragma unroll
      for (int i = 0; i < 4; ++i) o[m][i] = fmaf(sc, C[i], o[m][i]);
    };

    // ---- the interleaved stream: anomalous items, then normal items; value tile j rides
    // with key item j NK / 8 (all eight at once when there are no key items)
    Op mre[2], mim[2];
    uint2 E[2][2], O[2][2];
    uint2 asz[2][2];
    f4 Cv = zero;
    if (!HOP_SZ && NKA > 0) load_sz(0, asz[0][0], asz[0][1]);
    if (NKN > 0 && (HOP_SZ || NKA == 0)) load_meta(0, mre[0], mim[0]);
    if (DO_V) lookup(0, E[0], O[0]);
    __builtin_amdgcn_sched_barrier(0);
    constexpr int NSTEP = NK > 0 ? NK : 1;
#pragma unroll
    for (int k = 0; k < NSTEP; ++k) {
      if (k < NKA) {
        if (!HOP_SZ && k + 1 < NKA) load_sz(k + 1, asz[(k + 1) & 1][0], asz[(k + 1) & 1][1]);
        if (!HOP_SZ && k + 1 == NKA && NKN > 0) load_meta(0, mre[0], mim[0]);
        anomalous_item(k, asz[k & 1][0], asz[k & 1][1]);
      } else if (k < NK) {
        const int n = k - NKA;
        if (n + 1 < NKN) load_meta(n + 1, mre[(n + 1) & 1], mim[(n + 1) & 1]);
        normal_item(n, mre[n & 1], mim[n & 1]);
      }
      if (DO_V) {
#pragma unroll
        for (int j = 0; j < 8; ++j) {
          if ((NK > 0 ? (j * NK) / 8 : 0) == k) {
            if (j + 1 < 8) lookup(j + 1, E[(j + 1) & 1], O[(j + 1) & 1]);
            if (j > 0) add_tile(j - 1, Cv);
            Cv = value_tile(j, E[j & 1], O[j & 1]);
          }
        }
      }
      __builtin_amdgcn_sched_barrier(0);
    }
    if (DO_V) add_tile(7, Cv);
    cst = 0.0f;
    if (DO_K) {
      float cst_n = 0.0f;                        // non-FFT: sum over normal channels of q (z + s/2)
      if (U > 0 && !FFT) {
        // slot = token: the products are the scores' normal-channel part for my group
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          S[0][i] += accRe[i];
          S[1][i] += accIm[i];
        }
        cst_n = -fmaf(2.0f, accCn[0], accCs[0]);
      }
      if (IDFT && FULL) {
        // k-slot (kb, i) of the matrix against row 4 kb + i of the sums, one i at a time.  Coefficient 4 kb + i is
        // even where i is; from token t to t + 16 the even ones stay and the odd ones change their sign, so the
        // products for the first 16 tokens serve both halves
        const f4 Wr = __builtin_bit_cast(f4, w_tab[0][lane]), Wi = __builtin_bit_cast(f4, w_tab[2][lane]);
        f4 ev = zero, od = zero;
#pragma unroll
        for (int i = 0; i < 4; i += 2) {
          ev = __builtin_amdgcn_mfma_f32_16x16x4f32(Wr[i], accRe[i], ev, 0, 0, 0);
          od = __builtin_amdgcn_mfma_f32_16x16x4f32(Wr[i + 1], accRe[i + 1], od, 0, 0, 0);
          ev = __builtin_amdgcn_mfma_f32_16x16x4f32(Wi[i], accIm[i], ev, 0, 0, 0);
          od = __builtin_amdgcn_mfma_f32_16x16x4f32(Wi[i + 1], accIm[i + 1], od, 0, 0, 0);
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          S[0][i] += ev[i] + od[i];
          S[1][i] += ev[i] - od[i];
        }
      }
      if (IDFT && !FULL) {
        // split Y/16 into fp16 hi + lo, then the inverse DFT
        Op Yh, Yl, Wh[2], Wl[2];
        Wh[0].q = w_tab[0][lane]; Wh[1].q = w_tab[1][lane];
        Wl[0].q = w_tab[2][lane]; Wl[1].q = w_tab[3][lane];
#pragma unroll
        for (int i = 0; i < 4; i += 2) {
          const float r0 = accRe[i], r1 = accRe[i + 1];
          const float i0 = accIm[i], i1 = accIm[i + 1];
          Yh.u[i / 2] = pkrtz(r0, r1);
          Yh.u[2 + i / 2] = pkrtz(i0, i1);
          Yl.u[i / 2] = pkrtz(r0 - (float)Yh.v[i], r1 - (float)Yh.v[i + 1]);
          Yl.u[2 + i / 2] = pkrtz(i0 - (float)Yh.v[4 + i], i1 - (float)Yh.v[4 + i + 1]);
        }
#pragma unroll
        for (int mt = 0; mt < 2; ++mt) {
          S[mt] = mma(Wh[mt], Yh, S[mt]);
          S[mt] = mma(Wl[mt], Yh, S[mt]);
          S[mt] = mma(Wh[mt], Yl, S[mt]);
        }
      }
      if (UA > 0) cst = accC[0][0] + accC[1][0] + accC[2][0];                 // = -(sum q (z + 1.5 s)), 2 h times it like S and cst_n
      if (!FFT) cst -= cst_n;
    }
  };

  // the probabilities of the pair with masks (s0, s1), staged as [token][head] at stg: those of
  // its protected tokens go to the end of the list (lane = token; there is room for a pair)
  auto collect = [&](uint32_t s0, uint32_t s1, const uint8_t* stg) {
    uint32_t lane = tid & 63;
    asm volatile("" : "+v"(lane));
    const f4 va = *reinterpret_cast<const f4*>(stg + lane * 32), vb = *reinterpret_cast<const f4*>(stg + lane * 32 + 16);
    int pos = lpos + lcnt + (int)__builtin_amdgcn_mbcnt_hi(s1, __builtin_amdgcn_mbcnt_lo(s0, 0u));
    pos = pos >= LCAP ? pos - LCAP : pos;
    if (((lane < 32 ? s0 : s1) >> (lane & 31)) & 1u) {
      *reinterpret_cast<f4*>(&plist[wave][pos][0]) = va;
      *reinterpret_cast<f4*>(&plist[wave][pos][4]) = vb;
    }
    lcnt += __popc(s0) + __popc(s1);
  };
  // one batch: entries lfirst .. min(lcnt, BS) - 1 of the list against the rows in rowbuf (which
  // have landed), then the next batch's rows are requested.  Operand rows 0-7 are the heads'
  // probabilities rounded to fp16, rows 8-15 what the rounding left (FULL: times 2^18, so that the two
  // carry 22 bits down to 2^-14 of the running maximum, 22 to 11 down to 2^-25, 11 down to 2^-32 and none below 2^-43).
  auto batch = [&]() __attribute__((always_inline)) {   // (a call would put the running sums into memory)
    const int n = min(lcnt, BS);
    // lane numbers of its own, so that no address of a batch occupies a register between batches
    uint32_t ln = lane;
    asm volatile("" : "+v"(ln));
    const int x16 = ln & 15, kb = ln >> 4, hcol = x16 & 7, par = x16 >> 3;
    auto entry = [&](int idx) -> _Float16 {
      float v = plist[wave][lpos + idx][hcol];
      v = (unsigned)(idx - lfirst) < (unsigned)(n - lfirst) ? v : 0.0f;
      const _Float16 hi = (_Float16)v;
      return par ? (_Float16)(FULL ? (v - (float)hi) * 0x1p18f : v - (float)hi) : hi;
    };
    const float lo_row = FULL && (kb >> 1) ? 0x1p-18f : 1.0f;   // of my rows' products
    if (SAL == 1) {
      if (n < BS) {
        // rows without an entry count 0 times, and must not hold a NaN (a last batch only)
#pragma unroll
        for (int j = 0; j < BS / 4; ++j)
          if (4 * j + kb >= n) *reinterpret_cast<u32x4*>(&rowbuf[wave][j * 1024 + ln * 16]) = u32x4{0u, 0u, 0u, 0u};
        asm volatile("" ::: "memory");
      }
      h4 A;                                  // k-slots: rows 4 kb + i
#pragma unroll
      for (int i = 0; i < 4; ++i) A[i] = entry(4 * kb + i);
      // a transposing read hands lane x16 of kb the rows 4 kb .. 4 kb + 3 of channel 16 m + x16
      const int r = 4 * kb + (x16 >> 2);
      const uint32_t at = rowbuf_lds + r * 2 * D + (r & 7) * 32 + (x16 & 3) * 8;
      h4 Br[8];                              // all requested before the first is used
#pragma unroll
      for (int m = 0; m < 8; ++m)
        Br[m] = __builtin_bit_cast(h4, __builtin_amdgcn_ds_read_tr16_b64_v4i16(
            reinterpret_cast<__attribute__((address_space(3))) s16x4*>(at ^ (m * 32))));
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int m = 0; m < 8; ++m) {
        const h4 B = Br[m];
        if (FULL) {
          const f4 C = __builtin_amdgcn_mfma_f32_16x16x16f16(A, B, zero, 0, 0, 0);
#pragma unroll
          for (int i = 0; i < 4; ++i) o[m][i] = fmaf(lo_row, C[i], o[m][i]);
        } else {
          o[m] = __builtin_amdgcn_mfma_f32_16x16x16f16(A, B, o[m], 0, 0, 0);
        }
      }
    } else {
      const uint8_t* rec = &rowbuf[wave][0];
      Op A, one;                             // k-slots: rows kb + 4 i
#pragma unroll
      for (int i = 0; i < 8; ++i) A.v[i] = entry(kb + 4 * i);
#pragma unroll
      for (int i = 0; i < 4; ++i) one.u[i] = 0x3C003C00u;
      f4 P = mma(A, one, zero);
      if (FULL) P *= lo_row;
      // channel 16 m + x16 is field x16 % 4 of byte x16 / 4 of dword m of a row; the code stays where
      // it is: as an fp16 number code 2^(2 (x16 % 4) - 24), here times 2^15.  A row's dwords come four at a time
      // (a byte of a row at a time, 64 reads instead of 16: 28 layers x 6272 tokens, 20 % protected, 332 us a step; now 321)
      const uint32_t field = 0x00030003u << (2 * (x16 & 3));
      const uint32_t pick = 0x0C040C00u + 0x00010001u * (x16 >> 2);       // byte x16 / 4 of two rows into two halves
      const float unit = lo_row * ((float)(1 << 9) / (float)(1 << (2 * (x16 & 3))));
#pragma unroll
      for (int mq = 0; mq < 2; ++mq) {
        u32x4 w[8];
        _Float16 s4[4], z4[4];
#pragma unroll
        for (int i = 0; i < 8; ++i) w[i] = *reinterpret_cast<const u32x4*>(rec + (kb + 4 * i) * 32 + 16 * mq);
#pragma unroll
        for (int m = 0; m < 4; ++m) {
          s4[m] = reinterpret_cast<const _Float16*>(rec + 1024)[16 * (4 * mq + m) + x16];
          z4[m] = reinterpret_cast<const _Float16*>(rec + 1280)[16 * (4 * mq + m) + x16];
        }
        __builtin_amdgcn_sched_barrier(0);
        f4 C[4];
#pragma unroll
        for (int m = 0; m < 4; ++m) {
          Op B;
#pragma unroll
          for (int i = 0; i < 4; ++i)
            B.p[i] = bits_h2(__builtin_amdgcn_perm(w[2 * i + 1][m], w[2 * i][m], pick) & field) *
                     h2{(_Float16)32768.0f, (_Float16)32768.0f};
          C[m] = mma(A, B, zero);
        }
#pragma unroll
        for (int m = 0; m < 4; ++m) {
          const float sc = (float)s4[m] * unit, zc = (float)z4[m];
#pragma unroll
          for (int i = 0; i < 4; ++i) o[4 * mq + m][i] = fmaf(zc, P[i], fmaf(sc, C[m][i], o[4 * mq + m][i]));
        }
      }
    }
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");   // the rows have been read: their place may be refilled
    lpos = lpos + BS == LCAP ? 0 : lpos + BS;
    lcnt = max(0, lcnt - BS);
    lfirst = 0;
    rb += BS;
    fetch_rows();
  };

  // online softmax of the pair's scores: updates m_run, l_run (and rescales the running
  // sums and the listed probabilities when the maximum is raised), leaves the packed
  // probabilities in pp and, when the pair has protected tokens, stages them at stg as [token][head]
  // (first: no score came before, there is nothing to rescale)
  auto softmax = [&](auto first_c, const f4 (&S)[2], float cst, bool v1ok, bool stage_pl, uint8_t* stg) {
    constexpr bool FIRST = decltype(first_c)::value;
    // t = score - running maximum, in the exp2 domain, for my column at token slot i
    // (i < 4: token 4kb+i, else 16+4kb+i-4); a column without a group gets -inf
    const bool dead = par && !v1ok;
    const float c0 = dead ? -INFINITY : -cst * sc2;
    float c1 = FIRST ? c0 : c0 - m_run;
    float t[8];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      t[i] = fmaf(S[0][i], sc2, c1);
      t[4 + i] = fmaf(S[1][i], sc2, c1);
    }
    // The running maximum is raised lazily: only when some score exceeds it by more than 8
    // (p stays below 2^8), which needs no cross-lane traffic in the common case.
    float mx = fmaxf(fmaxf(fmaxf(t[0], t[1]), fmaxf(t[2], t[3])), fmaxf(fmaxf(t[4], t[5]), fmaxf(t[6], t[7])));
    if (FIRST) {
      const float smax = swap_max16(swap_max32(mx)), m_new = fmaxf(smax, from_xor8(smax));
#pragma unroll
      for (int i = 0; i < 8; ++i) t[i] -= m_new;
      m_run = m_new;
    } else if (__any(mx > 8.0f)) {
      // maximum over the 4 k-blocks and the 2 parities of the head (the first step has left a finite one)
      float smax = swap_max16(swap_max32(mx + m_run));
      smax = fmaxf(smax, from_xor8(smax));
      const float m_new = fmaxf(m_run, smax);
      const float shift = m_run - m_new, al = __builtin_amdgcn_exp2f(shift);
#pragma unroll
      for (int i = 0; i < 8; ++i) t[i] += shift;
      l_run *= al;
      m_run = m_new;
      // the PV accumulators are laid out by score-tile column as ROW 4kb + i
      if (kb == 0) al16[wave][x16] = al;
      float ar[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) ar[i] = al16[wave][4 * kb + i];
#pragma unroll
      for (int m = 0; m < 8; ++m)
#pragma unroll
        for (int i = 0; i < 4; ++i) o[m][i] *= ar[i];
      if ((SAL != 0)) {
        const f4 aa = *reinterpret_cast<const f4*>(&al16[wave][0]), ab = *reinterpret_cast<const f4*>(&al16[wave][4]);
        for (int e = lane; e < lcnt; e += 64) {
          const int pos = lpos + e >= LCAP ? lpos + e - LCAP : lpos + e;
          f4* l4 = reinterpret_cast<f4*>(&plist[wave][pos][0]);
          l4[0] *= aa;
          l4[1] *= ab;
        }
      }
    }
    float pr[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      pr[i] = __builtin_amdgcn_exp2f(t[i]);
    }
    l_run += ((pr[0] + pr[1]) + (pr[2] + pr[3])) + ((pr[4] + pr[5]) + (pr[6] + pr[7]));
    // probabilities as the A operand of P V (row = my column).  The k-slots of that product
    // are ordered (0,2), (4,6), (1,3), (5,7) in token-slot numbers: the order in which two
    // trit bytes expand (even slots, then odd slots).
    if (FULL) {
      // 24 bits = 3 x 8: the upper halves of p, of what they leave, and what is left then
      auto upper2 = [](float x, float y) -> uint32_t { return __builtin_amdgcn_perm(__float_as_uint(y), __float_as_uint(x), 0x07060302u); };
      auto rest = [](float x) -> float { return x - __uint_as_float(__float_as_uint(x) & 0xFFFF0000u); };
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int i = (r & 1) * 4 + (r >> 1);            // slots (0,2) (4,6) (1,3) (5,7)
        const float x1 = rest(pr[i]), y1 = rest(pr[i + 2]);
        pp[r] = upper2(pr[i], pr[i + 2]);
        pm[r] = upper2(x1, y1);
        pl[r] = upper2(rest(x1), rest(y1));
      }
    } else {
      pp[0] = pk_rne(pr[0], pr[2]);
      pp[1] = pk_rne(pr[4], pr[6]);
      pp[2] = pk_rne(pr[1], pr[3]);
      pp[3] = pk_rne(pr[5], pr[7]);
    }
    if ((SAL != 0) && stage_pl) {
      uint32_t ln = lane;
      asm volatile("" : "+v"(ln));
      const int kb = ln >> 4;
      float* pw = reinterpret_cast<float*>(stg) + (ln & 8) * 32 + (ln & 7);
#pragma unroll
      for (int i = 0; i < 8; ++i) pw[8 * slot_token(kb, i)] = pr[i];
    }
  };

  // ---------------- the loop, software-pipelined over two pairs: while the keys of pair p
  // are scored, the values (and protected rows) of the pair before it are added - two
  // independent chains of LDS reads, MFMAs and ALU work in one instruction stream.  A
  // pair's value records are therefore requested one step after its key records.
  // Step with key stage KS: keys of pair p in key stage KS; its values are requested into
  // value stage KS; the previous pair's are in KS ^ 1.  The probabilities of a pair with protected
  // tokens are staged where its keys were (nothing is requested into that stage before the next
  // step has collected them).
  static_assert(2 * KREC >= 64 * 8 * 4, "a pair's probabilities must fit its key stage");
  auto step = [&](auto ks_c, auto first_c) {
    constexpr int KS = decltype(ks_c)::value;
    constexpr bool FIRST = decltype(first_c)::value;
    const bool v1ok = (2 * p + 1) < a.ng;
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // keys of p, values of the pair before, rows of the batch
    if ((SAL != 0) && !FIRST && (sm0v | sm1v)) collect(sm0v, sm1v, ring_w + (KS ^ 1) * 2 * KREC);
    if ((SAL != 0) && !FIRST) {
      // one batch a step as a rule; more, each with a wait for its rows, when a pair brings many: until a pair's
      // 64 have room again.  (Here, where few registers are in use.  As one loop, the running sums changed
      // registers at every step, batch or not.)
      if (lcnt >= BS) batch();
      while (__builtin_expect(lcnt > LCAP - 64, 0)) {
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        batch();
      }
    }
    FirstHop hop;
    first_hop(ks_c, std::true_type{}, std::integral_constant<bool, !FIRST>{}, hop);
    __builtin_amdgcn_sched_barrier(0);
    fetch_keys(p + PSTEP, KS ^ 1, p + PSTEP < p_end);
    fetch_values(p, KS, !FIRST || !a.early);             // (early: requested at the start)
    // (the first rows here: in front of the operands of q, whose LDS reads then wait for the transfer, they cost
    // 0.4 us, at the end of the step 0.3)
    if (SAL != 0 && FIRST) fetch_rows();
    f4 S[2];
    float cst;
    scores_and_values(ks_c, std::true_type{}, std::integral_constant<bool, !FIRST>{}, hop, S, cst);
    softmax(first_c, S, cst, v1ok, (sm0c | sm1c) != 0, &ring[wave][0] + KS * 2 * KREC);
    if ((SAL != 0)) {
      sm0v = sm0c; sm1v = sm1c;
      sm0c = sm0n; sm1c = sm1n;
      load_masks(p + 2, sm0n, sm1n);
    }
  };
  int last_ks = -1;
  if (p < p_end) {
    step(std::integral_constant<int, 0>{}, std::true_type{});
    last_ks = 0;
    p += PSTEP;
    while (p < p_end) {
      step(std::integral_constant<int, 1>{}, std::false_type{});
      last_ks = 1;
      p += PSTEP;
      if (p >= p_end) break;
      step(std::integral_constant<int, 0>{}, std::false_type{});
      last_ks = 0;
      p += PSTEP;
    }
  }
  // the last pair's values
  if (last_ks >= 0) {
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    if ((SAL != 0) && (sm0v | sm1v)) collect(sm0v, sm1v, ring_w + last_ks * 2 * KREC);
    if ((SAL != 0) && lcnt > lfirst) batch();   // the rows of another batch arrive beside the values' products
    f4 S[2]; float cst;
    FirstHop hop;
    if (last_ks == 0) {
      first_hop(std::integral_constant<int, 1>{}, std::false_type{}, std::true_type{}, hop);
      scores_and_values(std::integral_constant<int, 1>{}, std::false_type{}, std::true_type{}, hop, S, cst);
    } else {
      first_hop(std::integral_constant<int, 0>{}, std::false_type{}, std::true_type{}, hop);
      scores_and_values(std::integral_constant<int, 0>{}, std::false_type{}, std::true_type{}, hop, S, cst);
    }
    if (SAL != 0) {
      while (lcnt > lfirst) {                  // what is left of the list
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        batch();
      }
    }
  }

  // ---------------- per-wave reduction
  // l: 4 k-blocks and 2 parities of each head
  l_run = swap_sum32(l_run);
  l_run = swap_sum16(l_run);
  l_run += from_xor8(l_run);
  // o: rows 4kb+i, (parity, head)
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");                // no transfer into the ring is left
  put_wave_sums(o, reinterpret_cast<float*>(&ring[wave][0]), x16, kb);
  if (kb == 0 && par == 0) { mw[hcol][wave] = m_run; lw[hcol][wave] = l_run; }
  __syncthreads();
  put_partial(a, split, kvh, b, tid, mw, lw, &ring[0][0], RING);
}

#undef VIDKV_DMA
#undef VIDKV_DMA_MORE

template <int NA8, bool TAIL>
static void launch_one(const AttnArgs& a, dim3 grid, hipStream_t st) {
  const int sal = a.n_s > 0 ? (a.sal_bits == 2 ? 2 : 1) : 0;
#define VIDKV_ATTN(S, F) hipLaunchKernelGGL((attn_mfma_kernel<NA8, S, F, TAIL>), grid, dim3(256), 0, st, a)
  if (a.use_fft) {
    if (sal == 2) VIDKV_ATTN(2, true); else if (sal == 1) VIDKV_ATTN(1, true); else VIDKV_ATTN(0, true);
  } else {
    if (sal == 2) VIDKV_ATTN(2, false); else if (sal == 1) VIDKV_ATTN(1, false); else VIDKV_ATTN(0, false);
  }
#undef VIDKV_ATTN
}

}  // namespace vidkv
