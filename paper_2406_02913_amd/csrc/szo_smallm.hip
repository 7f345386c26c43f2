// Few-token path (16 or 32 token rows per pass; the host slices up to 128 tokens): the forward is bound by
// streaming the 4-bit weights from HBM, not by the matrix cores, and the paper's own guideline for this regime (Appendix C.5) is the
// SparseAddMM association:   y = x Dequantize(Q(w_dense))^T  +  x w_sparse^T.
// Two consequences shape this kernel:
//   * the dense product does not depend on the perturbation, so ONE pass over the weights
//     serves both the +eps and the -eps forward of a ZO step (Definition 1 needs f at both);
//   * the sparse weights are  v +- eps z  (Section 3.4), so the sparse product splits into
//     a = x v^T  (added to the dense part) and  b = x z^T:  y(+-) = dense + a +- eps b.
//
// One workgroup = 256 output columns (4 bands of 64 rows of W, one wave each) x all of K, walked in
// chunks of 256 columns of x that are staged in LDS as fp16 (16 or 32 token rows, zero padded).  The
// kernel is written for several small waves per SIMD (~150 registers, ~30 KB of LDS per workgroup):
// a streaming-read probe on this chip reaches its ceiling with a few 16-byte loads in flight per
// wave as long as enough waves are resident, and the resident waves hide each other's stalls.
// Per chunk a wave
//   - streams its band's codes, 16 bytes per lane, one 128-column block ahead, and turns them in registers into
//     the B operand of v_mfma_f32_16x16x32_f16 (no LDS round trip: every weight is used once).
//     With a quantisation group of 128 the codes are NOT re-centred: 0x6400|c reads 1024+c and
//     0x5400|(c<<4) reads 64+c, both exact in fp16, and the constant part
//     sum_k x[m,k] (1032 | 72) of each 128-column block comes out of one more MFMA chain per block
//     against a constant operand and seeds the chains of the block's four subtiles, negated.  The
//     block's partial product then takes the group scale in fp32.
//   - keeps a ring of its band's sensitive entries in LDS (position, fp16 v, fp16 z; z from the
//     same Philox/Box-Muller routine and counters as the large-batch kernel and the update, 256
//     entries per refill so that all lanes work), and multiplies them in groups of 16 entries as a
//     second, tiny MFMA: A = the entries' columns of x (gathered from LDS), B = a one-hot matrix
//     that routes entry e to its row (value v or z).  No atomics, no read-modify-write chains.
// The epilogue forms y(+-), stores y for the requested sign and folds the squared error against the
// target into two fp64 partials per workgroup (one per sign); a launch asks for either or both.
// Everything is accumulated in a fixed order: results are bit-reproducible.
#include <algorithm>
#include <cstddef>
#include <type_traits>
#include <utility>
#include <vector>
#include "szo_few.h"

namespace szo {

constexpr int SM_BN = 256;              // output columns per workgroup = 4 bands of 64
constexpr int SM_KC = 256;              // columns of x staged per chunk (double buffered) = 2 blocks of 128
constexpr int SM_XSTRIDE = SM_KC + 8;   // LDS row stride of x in fp16 elements (+16 B against bank conflicts)
constexpr int SM_WIN = 256;             // sensitive entries computed per refill (4 per lane)
constexpr int SM_CAP = 512;             // entries held per band (ring)
#ifndef SM_MIN_BLOCKS
#define SM_MIN_BLOCKS 4                 // workgroups per CU the register budget of a 16-row pass is set for (<= 128 registers, no spills;
                                        // the table format keeps its tables in 32 more registers: three workgroups)
#endif

// Position of column kk inside its 8-element chunk in LDS: chunks keep the order 0,4,1,5,2,6,3,7
// in which the dequantised nibbles come out, so that x and the weights pair up element by element.
__device__ __forceinline__ int sm_xpos(int kk) {
  const int w = kk & 7;
  return (kk & ~7) | ((w & 3) << 1) | (w >> 2);
}

// MODE 1 (uniform format, quantisation group of 128): the scales of a block's four subtiles are
// prefetched with one 8-byte load and applied to each block's partial product, and the codes stay
// un-centred as described at the top.  MODE 0 (the other group sizes): the scale is read from memory
// where it is needed and applied to every element before the product (a plain, slower path).
// MODE 2 (table format): dq = lut[row][code]; a lane keeps the tables of its four rows in registers
// (32 of them; it needs neither scales nor the constants of the un-centred codes, so it still fits
// the register budget of three workgroups per CU).
// R = 16-row blocks of tokens per pass (1, 2 or 3).  With R > 1 every dequantised operand is multiplied
// with R blocks of token rows, so that matrices with more than 16 tokens stream their weights less
// often; each block costs 48 more registers (accumulators and activation operands): 196 and 253
// registers, i.e. two workgroups per CU instead of three.
// DUAL (R = 2 only): the two forwards read different activations (x for +eps, x2 for -eps).  Block 0 then
// holds 16 token rows of x and block 1 the same rows of x2: still one pass over the weights for both
// signs, but nothing else is shared, and y(+) = acc[0] + eps accz[0], y(-) = acc[1] - eps accz[1].
// ONCE: the codes are loaded as a non-temporal stream.  The host chooses it for launches that read every byte of
// their codes exactly once (one slice per strip) and stream more of them than the chip's last-level cache
// holds: they then do not displace what IS re-read -- the activations (by every strip of a matrix), the sparse
// values (by the update that follows).  Measured on a 32-block 7B-shaped stack at 16 tokens: 625 -> 592 us per
// launch, update 23.3 -> 21.3 us.  With several slices the slices of a strip share the codes through the L2
// and the hint costs 2 % (64 tokens) to 10 % (224 tokens); a stack that fits the last-level cache (one or two
// decoder blocks) is re-read from there step after step and loses 6 % with the hint: plain loads in both
// cases.  (A run-time choice between the two loads is folded into one plain load by the compiler, hence a
// template parameter.)
template <int MODE, int R, bool DUAL = false, bool ONCE = false>
__global__ void __launch_bounds__(256, R == 1 ? (MODE == SM_LUT ? 3 : SM_MIN_BLOCKS) : 2) small_m_kernel(SmallArgs a) {
  static_assert(R >= 1 && R <= 3, "one to three blocks of 16 token rows");
  static_assert(!DUAL || R == 2, "two activation sets: one block of rows each");
  constexpr bool FAST = MODE == SM_FAST, LUT = MODE == SM_LUT;
  constexpr int ROWS = SM_ROWS * R;                          // rows of activations staged per pass
  constexpr int TOK = DUAL ? SM_ROWS : ROWS;                 // token rows of one pass
  extern __shared__ __attribute__((aligned(16))) uint8_t smem[];
  _Float16* const xs = reinterpret_cast<_Float16*>(smem);                        // [2][ROWS][SM_XSTRIDE]
  uint16_t* const winp = reinterpret_cast<uint16_t*>(xs + 2 * ROWS * SM_XSTRIDE);      // [4 bands][SM_CAP] packed position (see refill)
  uint16_t* const winv = winp + 4 * SM_CAP;                                        // fp16 bits of v
  uint16_t* const winz = winv + 4 * SM_CAP;                                        // fp16 bits of z

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  int bid = xcd_unit((int)blockIdx.x, (int)gridDim.x);
  // ---- which slice of token rows, which matrix, which 256-column strip ----
  // Consecutive (remapped) ids are the slices of one strip: they read the same weights, so they should
  // run at the same time on the same XCD and share them through its L2.
  const int slice = bid % a.slices;
  bid /= a.slices;
  SmallMat mt = find_matrix(a, bid);
  // a launch has as many slices of TOK token rows per strip as its longest matrix needs
  if (slice * TOK >= mt.M) return;
  mt.x += (size_t)slice * TOK * (size_t)mt.K;
  if (DUAL) mt.x2 += (size_t)slice * TOK * (size_t)mt.K;
  if (mt.target) mt.target += (size_t)slice * TOK * (size_t)mt.N;
  if (mt.y) mt.y += (size_t)slice * TOK * (size_t)mt.N;
  mt.M = min(TOK, mt.M - slice * TOK);
  mt.partial_base += slice * ((mt.N + SM_BN - 1) / SM_BN);      // slice i of a matrix: partials [i * strips ..)
  const auto g_x = SZO_GLOBAL(uint16_t, mt.x);
  const auto g_x2 = SZO_GLOBAL(uint16_t, DUAL ? mt.x2 : mt.x);
  const auto g_q = SZO_GLOBAL(uint8_t, mt.qweight);
  const auto g_scales = SZO_GLOBAL(uint16_t, mt.scales);
  const auto g_tile_ptr = SZO_GLOBAL(uint32_t, mt.tile_ptr);
  const auto g_sp_idx = SZO_GLOBAL(uint32_t, mt.sp_idx);
  const auto g_sp_val = SZO_GLOBAL(float, mt.sp_val);
  const auto g_target = SZO_GLOBAL(uint16_t, mt.target);
  float __attribute__((address_space(1)))* const g_y = (float __attribute__((address_space(1)))*)mt.y;
  const int strip = bid - mt.first_block;
  const int n0 = strip * SM_BN;
  const int N = mt.N, K = mt.K, M = mt.M;
  const int ktiles = K >> 6;
  const int band = (n0 >> 6) + wave;                        // band of the sparse layout owned by this wave
  const bool band_ok = band * 64 < N && mt.nnz > 0;
  const int nn = lane & 15, jj = lane >> 4;                 // B operand: column nn of a 16-column subtile, k-group jj
  const int nchunks = (K + SM_KC - 1) / SM_KC;
  const int nkb_total = K >> 7;

  uint32_t magic_lo = 0x64006400u, magic_hi = 0x54005400u;
  asm volatile("" : "+v"(magic_lo), "+v"(magic_hi));
  // B operand of the constant-part chain: every column holds -(1032, 1032, 72, 72, 1032, 1032, 72, 72), the
  // offsets of the un-centred codes in the element order (0,4)(1,5)(2,6)(3,7)
  const half8_t minus_offsets = {(_Float16)-1032.0f, (_Float16)-1032.0f, (_Float16)-72.0f, (_Float16)-72.0f,
                                 (_Float16)-1032.0f, (_Float16)-1032.0f, (_Float16)-72.0f, (_Float16)-72.0f};

  uint16_t* const my_winp = winp + wave * SM_CAP;
  uint16_t* const my_winv = winv + wave * SM_CAP;
  uint16_t* const my_winz = winz + wave * SM_CAP;

  float4_t acc[R][4], accz[R][4];                           // per block of 16 token rows: dense + x v^T ;  x z^T
#pragma unroll
  for (int rb = 0; rb < R; ++rb)
#pragma unroll
    for (int s = 0; s < 4; ++s) { acc[rb][s] = float4_t{0.0f, 0.0f, 0.0f, 0.0f}; accz[rb][s] = float4_t{0.0f, 0.0f, 0.0f, 0.0f}; }

  // Banded layout (see the header): the band's 64 rows of one 64-column tile are 2 KB in a row, so
  // the 16 rows x 32 bytes that the lanes of one k-group pair read are contiguous, and a lane's four
  // scales of a group (rows nn, nn+16, nn+32, nn+48) are 8 bytes in a row.  Bands past N re-read the
  // last band: their outputs are never used.  32-bit byte offsets from the uniform base pointers
  // take half the registers of per-lane pointers.
  const uint32_t bsafe = (uint32_t)min(band, (N + 63) / 64 - 1);
  uint32_t qoff[4];
#pragma unroll
  for (int s = 0; s < 4; ++s)
    qoff[s] = (bsafe * (uint32_t)ktiles * 64u + (uint32_t)(16 * s + nn)) * 32u + (uint32_t)(jj >> 1) * 2048u + (uint32_t)(jj & 1) * 16u;
  const int gshift = mt.group_shift;
  const uint32_t soff = (bsafe * (uint32_t)(K >> gshift) * 64u + (uint32_t)nn * 4u) * 2u;
  // table format: the tables of rows nn, nn+16, nn+32, nn+48 of the band (mt.scales is the table array);
  // rows past N re-read the last row's table, their outputs are never used
  uint32_t tb[LUT ? 4 : 1][8];
  if (LUT) {
#pragma unroll
    for (int s = 0; s < (LUT ? 4 : 1); ++s) {
      const int n = min((int)bsafe * 64 + 16 * s + nn, N - 1);
      load_lut_planes(g_scales + (size_t)n * 16, tb[s]);
    }
  }
  // ---- x staging: piece = 8 columns (16 bytes of bf16) of one row; thread handles pieces
  //      (row tid>>5, columns 8*(tid&31)..) and the same columns of rows 8 i + (tid>>5), i < 2 R ----
  // Loads are unconditional, from clamped addresses, and out-of-range parts are zeroed only when the
  // registers are stored to LDS: a branch or an early use here would make every later wait a full drain.
  u32x4 xr[2 * R];
  auto load_x = [&](int c) {
    const int col = min(c * SM_KC + 8 * (tid & 31), K - 8);
#pragma unroll
    for (int i = 0; i < 2 * R; ++i) {
      const int row = (tid >> 5) + 8 * i;                   // DUAL: staged rows 16.. are token rows 0.. of x2
      const int m = min(DUAL ? (row & 15) : row, M - 1);
      xr[i] = *reinterpret_cast<const u32x4 __attribute__((address_space(1)))*>(((DUAL && i >= 2) ? g_x2 : g_x) + (size_t)m * K + col);
    }
  };
  auto store_x = [&](int c) {
    const int ch = tid & 31, buf = c & 1;
    const bool col_ok = c * SM_KC + 8 * ch < K;
#pragma unroll
    for (int i = 0; i < 2 * R; ++i) {
      const int m = (tid >> 5) + 8 * i;
      const bool ok = col_ok && (DUAL ? (m & 15) : m) < M;
      u32x4 o;
#pragma unroll
      for (int w = 0; w < 4; ++w) o[w] = ok ? sm_stage_x_word(xr[i], w) : 0u;
      *reinterpret_cast<u32x4*>(xs + (buf * ROWS + m) * SM_XSTRIDE + 8 * ch) = o;
    }
  };

  // ---- code stream: slot kbl*4+s holds subtile s of the chunk's 128-column block kbl ----
#ifndef SM_RING
#define SM_RING 1                       // 128-column blocks of codes in flight per wave (1 or 2)
#endif
  // slot (b % SM_RING)*4 + s: subtile s of 128-column block b.  With two blocks in flight the stream
  // keeps running while the wave is busy with the sparse part and the barrier of a chunk.
  constexpr int RING = SM_RING;             // (two blocks in flight measured no faster with R = 2 either)
  u32x4 qbuf[4 * RING];
  auto load_q = [&](int slot, int gkb) {
    const auto* src = reinterpret_cast<const u32x4 __attribute__((address_space(1)))*>(g_q + (size_t)min(gkb, nkb_total - 1) * 4096 + qoff[slot & 3]);
    qbuf[slot] = ONCE ? __builtin_nontemporal_load(src) : *src;
  };
#pragma unroll
  for (int i = 0; i < 4 * RING; ++i) load_q(i, i >> 2);
  u32x2 sc[2] = {u32x2{0u, 0u}, u32x2{0u, 0u}};             // FAST: block kbl of the chunk: the lane's four scales (s = 0..3)
  auto load_scales = [&](int c) {
#pragma unroll
    for (int kbl = 0; kbl < 2; ++kbl)
      sc[kbl] = *reinterpret_cast<const u32x2 __attribute__((address_space(1)))*>(
          reinterpret_cast<const uint8_t __attribute__((address_space(1)))*>(g_scales) +
          (size_t)min(2 * c + kbl, nkb_total - 1) * 128 + soff);
  };
  if (FAST) load_scales(0);
  load_x(0);

  // ---- sensitive entries of this band: boundaries per chunk, ring of entries in LDS ----
  auto tp_at = [&](int c) -> uint32_t {                     // first entry of the band at or after chunk c
    return band_ok ? g_tile_ptr[(uint32_t)band * (uint32_t)ktiles + (uint32_t)min(c * (SM_KC / 64), ktiles)] : 0u;
  };
  uint32_t tp0 = tp_at(0), tp1 = tp_at(1);
  uint32_t w_hi = __builtin_amdgcn_readfirstlane(tp0) & ~3u;      // entries below w_hi have been generated
  // A refill is only reached with band_ok (some entry of the band is wanted), so nnz > 0 there.  Its
  // loads are issued where they are used: refills are rare (256 entries each) and the other resident
  // waves cover the wait, while holding the values across the dense loop would cost 8 registers.
  auto refill = [&]() {
    const uint32_t j = w_hi + 4u * lane;
    uint32_t pf_idx[4];
    float pf_val[4];
    {
      const uint32_t last = mt.nnz - 1u;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const uint32_t je = min(j + e, last);               // clamped; entries past the end are never consumed
        pf_idx[e] = g_sp_idx[je];
        pf_val[e] = g_sp_val[je];
      }
    }
    float z[4] = {0.0f, 0.0f, 0.0f, 0.0f};
    if (a.eps != 0.0f) zbar_quad((mt.nnz_base + j) >> 2, a.seed, a.step, z);
    uint32_t p[4];
    half4_t vh, zh;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const uint32_t flat = pf_idx[e];
      const uint32_t n = sm_fast_div(flat, mt.div_mul, mt.div_shift);
      const uint32_t r = n - (uint32_t)(band * 64);
      const uint32_t k = flat - n * (uint32_t)K;
      // window word: bits 0-7 position of the column inside the staged chunk row, 8-11 row mod 16, 12-13 subtile
      p[e] = (uint32_t)sm_xpos((int)(k & (uint32_t)(SM_KC - 1))) | ((r & 15u) << 8) | (((r >> 4) & 3u) << 12);
      vh[e] = (_Float16)pf_val[e];
      zh[e] = (_Float16)z[e];
    }
    const uint32_t ring = j & (uint32_t)(SM_CAP - 1);
    *reinterpret_cast<u32x2*>(my_winp + ring) = u32x2{p[0] | (p[1] << 16), p[2] | (p[3] << 16)};
    *reinterpret_cast<u32x2*>(my_winv + ring) = __builtin_bit_cast(u32x2, vh);
    *reinterpret_cast<u32x2*>(my_winz + ring) = __builtin_bit_cast(u32x2, zh);
    w_hi += SM_WIN;
  };

  store_x(0);
  __syncthreads();

  for (int c = 0; c < nchunks; ++c) {
    const int kc = c * SM_KC;
    const _Float16* const xc = xs + (c & 1) * ROWS * SM_XSTRIDE;
    const uint32_t tp2 = tp_at(c + 2);
    // next chunk's x: requested before the dense part, so that it has landed when the (short) sparse part
    // is over and store_x wants it (two blocks of rows: 64 tokens 1.547 -> 1.535 ms; one block measured no gain,
    // and with three there are no registers to hold it that long)
    constexpr bool EARLY_X = R == 2;
    if (EARLY_X) load_x(min(c + 1, nchunks - 1));           // the last chunk re-reads itself; never stored

    // ---- dense: stream this band's codes ----
#pragma unroll
    for (int kbl = 0; kbl < 2; ++kbl) {
      // blocks past the end of K multiply clamped codes with the zeros staged for x: no branch needed
      // R = 1: the activation operands are read from LDS where they are used (16 registers less, which is
      // what lets four workgroups share a CU); with more blocks of rows they are read once per block.
      constexpr bool AF_LATE = R == 1;
      auto read_af = [&](int rb, int t) {
        return *reinterpret_cast<const half8_t*>(xc + (16 * rb + nn) * SM_XSTRIDE + kbl * 128 + 32 * jj + 8 * t);
      };
      half8_t af[AF_LATE ? 1 : R][AF_LATE ? 1 : 4];
      if (!AF_LATE) {
#pragma unroll
        for (int rb = 0; rb < R; ++rb)
#pragma unroll
          for (int t = 0; t < 4; ++t) af[rb][t] = read_af(rb, t);
      }
      auto af_of = [&](int rb, int t) { return AF_LATE ? read_af(rb, t) : af[AF_LATE ? 0 : rb][AF_LATE ? 0 : t]; };
      // FAST: minus the constant part of the un-centred codes, sum_k x[m,k] (1032 | 72) over the block, from
      // one more MFMA chain against a constant operand; it seeds the four subtiles' chains.
      float4_t init[R];
#pragma unroll
      for (int rb = 0; rb < R; ++rb) {
        init[rb] = float4_t{0.0f, 0.0f, 0.0f, 0.0f};
        if (FAST) {
#pragma unroll
          for (int t = 0; t < 4; ++t) init[rb] = __builtin_amdgcn_mfma_f32_16x16x32_f16(af_of(rb, t), minus_offsets, init[rb], 0, 0, 0);
        }
      }
#pragma unroll
      for (int s = 0; s < 4; ++s) {
        constexpr int kRingMask = RING - 1;
        const int slot = (kbl & kRingMask) * 4 + s;
        const u32x4 q = qbuf[slot];
        load_q(slot, 2 * c + kbl + RING);                   // the slot is free: fetch the block RING ahead
        _Float16 sh = (_Float16)0.0f;
        if (FAST) {
          sh = __builtin_bit_cast(half4_t, sc[kbl])[s];
        } else if (!LUT) {
          const uint32_t gi = (uint32_t)min((kc + kbl * 128 + 32 * jj) >> gshift, (K >> gshift) - 1);
          sh = __builtin_bit_cast(_Float16, *reinterpret_cast<const uint16_t __attribute__((address_space(1)))*>(
              reinterpret_cast<const uint8_t __attribute__((address_space(1)))*>(g_scales) + (size_t)gi * 128 + soff + 2 * s));
        }
        const half2_t s2 = {sh, sh};
        float4_t tmp[R];
#pragma unroll
        for (int rb = 0; rb < R; ++rb) tmp[rb] = init[rb];
#pragma unroll
        for (int t = 0; t < 4; ++t) {
          const half8_t b = LUT ? sm_lut_word(q[t], tb[LUT ? s : 0]) : sm_dequant_word<FAST>(q[t], magic_lo, magic_hi, s2);
#pragma unroll
          for (int rb = 0; rb < R; ++rb) tmp[rb] = __builtin_amdgcn_mfma_f32_16x16x32_f16(af_of(rb, t), b, tmp[rb], 0, 0, 0);
        }
#pragma unroll
        for (int rb = 0; rb < R; ++rb) {
          if (FAST) {
            const float sf = (float)sh;                      // column nn of the subtile: the lane's own row of W
#pragma unroll
            for (int r = 0; r < 4; ++r) acc[rb][s][r] = fmaf(tmp[rb][r], sf, acc[rb][s][r]);
          } else {
#pragma unroll
            for (int r = 0; r < 4; ++r) acc[rb][s][r] += tmp[rb][r];
          }
        }
        // keep the subtiles in program order: hoisting the later ones' loads and unpacking costs registers,
        // and the latency they would hide is covered by the other resident waves
        __builtin_amdgcn_sched_barrier(0);
      }
    }

    // next chunk's x and scales: requested now that this chunk's are no longer needed, landing
    // while the sparse part runs
    if (!EARLY_X) load_x(min(c + 1, nchunks - 1));
    if (FAST) load_scales(c + 1);                           // clamped inside

    // ---- sparse: this band's entries inside the chunk, 16 at a time (4 per k-group of the MFMA) ----
    {
      const uint32_t j_lo = __builtin_amdgcn_readfirstlane(tp0), j_hi = __builtin_amdgcn_readfirstlane(tp1);
      const uint32_t span = j_hi - j_lo;
      const _Float16* const xrow = xc + nn * SM_XSTRIDE;
      for (uint32_t g0 = j_lo & ~3u; g0 < j_hi; g0 += 16u) {
        // refilling here never overwrites an entry at or above g0: w_hi < g0 + 16 and SM_WIN + 16 <= SM_CAP
        while (w_hi < min(g0 + 16u, j_hi)) refill();
        const uint32_t e0 = g0 + 4u * (uint32_t)jj;
        const uint32_t ring = e0 & (uint32_t)(SM_CAP - 1);
        const u32x2 pw = *reinterpret_cast<const u32x2*>(my_winp + ring);
        const u32x2 vw = *reinterpret_cast<const u32x2*>(my_winv + ring);
        const u32x2 zw = *reinterpret_cast<const u32x2*>(my_winz + ring);
        const uint32_t rel = e0 - j_lo;                      // wraps for entries before the chunk's first
        half4_t ax[R];
        uint32_t mlo[4], mhi[4];                            // entry i: 0xFFFF in halfword s of (mlo, mhi) iff this lane
#pragma unroll                                              // owns the entry's row in subtile s
        for (int i = 0; i < 4; ++i) {
          const uint32_t w = pw[i >> 1];
          const int sh = 16 * (i & 1);
          // Entries outside [j_lo, j_hi) are masked out below; their column field is < 256 whatever the
          // window holds, so the gather stays inside the staged row.
          const uint32_t col = __builtin_amdgcn_ubfe(w, sh, 8);
#pragma unroll
          for (int rb = 0; rb < R; ++rb) ax[rb][i] = xrow[16 * rb * SM_XSTRIDE + col];
          const bool mine = rel + (uint32_t)i < span && __builtin_amdgcn_ubfe(w, sh + 8, 4) == (uint32_t)nn;
          const uint32_t s16 = (w >> (sh + 8)) & 0x30u;     // 16 * subtile
          const uint64_t m = (uint64_t)0xFFFFu << s16;
          mlo[i] = mine ? (uint32_t)m : 0u;
          mhi[i] = mine ? (uint32_t)(m >> 32) : 0u;
        }
#pragma unroll
        for (int s = 0; s < 4; ++s) {
          u32x2 bv, bz;
#pragma unroll
          for (int h = 0; h < 2; ++h) {
            const uint32_t ma = (s < 2) ? mlo[2 * h] : mhi[2 * h], mb = (s < 2) ? mlo[2 * h + 1] : mhi[2 * h + 1];
            // halfword (s & 1) of ma -> low half, of mb -> high half
            const uint32_t mask = __builtin_amdgcn_perm(mb, ma, (s & 1) ? 0x07060302u : 0x05040100u);
            bv[h] = vw[h] & mask;
            bz[h] = zw[h] & mask;
          }
#pragma unroll
          for (int rb = 0; rb < R; ++rb) {
            acc[rb][s] = __builtin_amdgcn_mfma_f32_16x16x16f16(ax[rb], __builtin_bit_cast(half4_t, bv), acc[rb][s], 0, 0, 0);
            accz[rb][s] = __builtin_amdgcn_mfma_f32_16x16x16f16(ax[rb], __builtin_bit_cast(half4_t, bz), accz[rb][s], 0, 0, 0);
          }
        }
      }
    }
    tp0 = tp1; tp1 = tp2;

    if (c + 1 < nchunks) store_x(c + 1);
    __syncthreads();                                        // next chunk's x complete; this chunk's no longer read
  }

  // ---- epilogue: accumulator (rb, s), register r = token row 16*rb + 4*jj + r, column 16*s + nn of the band ----
  double lp = 0.0, lm = 0.0;
#pragma unroll
  for (int rb = 0; rb < R; ++rb)
#pragma unroll
  for (int s = 0; s < 4; ++s) {
    const int nl = 16 * s + nn, n = n0 + wave * 64 + nl;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int m = (DUAL ? 0 : 16 * rb) + 4 * jj + r;     // token row
      if (m < M && n < N) {
        const float pz = a.eps * accz[rb][s][r];
        const float yp = acc[rb][s][r] + pz, ym = acc[rb][s][r] - pz;
        if (a.loss_mode) {
          const float t = __uint_as_float((uint32_t)g_target[(size_t)m * N + n] << 16);
          const float dp = yp - t, dm = ym - t;
          if (!DUAL || rb == 0) lp += (double)(dp * dp);    // DUAL: block 0 is the +eps forward, block 1 the -eps one
          if (!DUAL || rb == 1) lm += (double)(dm * dm);
        }
        if (!DUAL && a.store_sign) g_y[(size_t)m * N + n] = a.store_sign > 0 ? yp : ym;
      }
    }
  }
  if (a.loss_mode) {
    __shared__ double red[2][4];
    lp = wave_sum(lp);
    lm = wave_sum(lm);
    if (lane == 0) { red[0][wave] = lp; red[1][wave] = lm; }
    __syncthreads();
    if (tid == 0) {
      const int pi = mt.partial_base + strip;
      ((double __attribute__((address_space(1)))*)a.partial_plus)[pi] = ((red[0][0] + red[0][1]) + (red[0][2] + red[0][3])) * mt.loss_scale;
      ((double __attribute__((address_space(1)))*)a.partial_minus)[pi] = ((red[1][0] + red[1][1]) + (red[1][2] + red[1][3])) * mt.loss_scale;
    }
  }
}

// Sparse ZO-SGD update of every matrix of a table in one launch (Section 3.4, fixed-parameter
// update rule): thread = one Philox counter = four consecutive entries of one matrix.  A matrix's
// counters start at a multiple of 64 threads, so a wave serves one matrix: it finds the table entry by
// a binary search on scalar loads (through the constant address space) and keeps the entry's fields in
// scalar registers.  (Searching per lane with vector loads made every wave wait for eight dependent
// memory round trips before it could touch its entries; the launch then took 27 us for 52 MB.)
struct UpdateArgs {
  const SmallMat* table;    // as in SmallArgs
  int n_mats;
  int partials_per_sign;    // > 0: the losses are still partials, and this launch forms g from them
  const double* partials;   // "+" partials, then "-" partials
  double* scalars;          // (L+, L-, g): written if partials_per_sign > 0, else g is read
  int64_t total_quads;
  uint64_t seed, step;
  float lr, eps;
};
struct InlineUpdateArgs { UpdateArgs staged; SmallMat inl[kInlineMats]; };         // the table in the kernel arguments

// What reduce_step_kernel adds up, in its order: 256 threads stand for its 1024.  Both signs side by side, as there.
__device__ __forceinline__ void block_sums_as_1024(const double* __restrict__ v, int count, double (&scratch)[2][16], double (&total)[2]) {
  double a[4][2][4] = {};
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    int i = 256 * k + (int)threadIdx.x;
    for (; i + 3 * 1024 < count; i += 4 * 1024)
#pragma unroll
      for (int c = 0; c < 4; ++c)
        for (int s = 0; s < 2; ++s) a[k][s][c] += v[s * count + i + 1024 * c];
    for (; i < count; i += 1024)
      for (int s = 0; s < 2; ++s) a[k][s][0] += v[s * count + i];
  }
#pragma unroll
  for (int k = 0; k < 4; ++k)
#pragma unroll
    for (int s = 0; s < 2; ++s) {
      const double w = wave_sum((a[k][s][0] + a[k][s][1]) + (a[k][s][2] + a[k][s][3]));
      if ((threadIdx.x & 63) == 0) scratch[s][4 * k + (threadIdx.x >> 6)] = w;
    }
  __syncthreads();
#pragma unroll
  for (int s = 0; s < 2; ++s) {
    total[s] = 0.0;
    for (int i = 0; i < 16; ++i) total[s] += scratch[s][i];
  }
}

// With few partials every workgroup adds them up by itself (same order, same g everywhere) instead of waiting for a
// launch that does: a step over one 256 x 256 layer at 64 tokens has 16 of them per sign.
// REDUCE and the inline table are compile-time: the update of a stack is bound by how many waves are resident while their
// table search, Philox rounds and value loads follow each other, and keeps the small form (21 registers, no LDS, 8 waves per
// SIMD).  As one kernel for everything (74 registers, 6 waves) it took 22.8 / 24.6 / 25.3 us on 32 OPT blocks at 1 / 16 / 64
// tokens instead of 20.7 / 22.3 / 22.5.
template <bool REDUCE, typename Args>
__global__ void __launch_bounds__(256) sparse_update_table_kernel(Args args) {
  constexpr bool INLINE = std::is_same_v<Args, InlineUpdateArgs>;
  const UpdateArgs& a = reinterpret_cast<const UpdateArgs&>(args);
  static_assert(offsetof(InlineUpdateArgs, staged) == 0, "both forms begin alike");
  constexpr int W = (int)(sizeof(SmallMat) / 4), FQ = (int)(offsetof(SmallMat, first_quad) / 4);
  static_assert(offsetof(SmallMat, first_quad) % 8 == 0, "first_quad is read as two words");
  const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  const int64_t tw = (int64_t)blockIdx.x * 256 + 64 * wave;           // the wave's first thread
  if (!REDUCE && tw >= a.total_quads) return;
  // z and the values first: what g waits for (the sums of the losses) is a chain of its own
  const uint64_t seed = a.seed, step = a.step;
  typedef const uint32_t __attribute__((address_space(4)))* words;
  const words tab = INLINE ? (words)__builtin_amdgcn_kernarg_segment_ptr() + offsetof(InlineUpdateArgs, inl) / 4 : (words)a.table;
  int lo = 0, hi = a.n_mats - 1;                                      // last matrix whose first_quad <= tw
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    const int64_t fq = (int64_t)(((uint64_t)tab[mid * W + FQ + 1] << 32) | tab[mid * W + FQ]);
    if (fq <= tw) lo = mid; else hi = mid - 1;
  }
  struct Words { uint32_t w[W]; } raw;
#pragma unroll
  for (int i = 0; i < W; ++i) raw.w[i] = tab[lo * W + i];
  const SmallMat mt = __builtin_bit_cast(SmallMat, raw);
  const int64_t tq = tw + (int64_t)(threadIdx.x & 63) - mt.first_quad, j0 = 4 * tq;
  const bool mine = tw < a.total_quads && j0 < (int64_t)mt.nnz, whole = mine && j0 + 4 <= (int64_t)mt.nnz;
  if (!REDUCE && !mine) return;
  float z[4] = {0.0f, 0.0f, 0.0f, 0.0f};
  float __attribute__((address_space(1)))* const v = (float __attribute__((address_space(1)))*)mt.sp_val + j0;
  typedef float f32x4 __attribute__((ext_vector_type(4)));
  f32x4 w = {0.0f, 0.0f, 0.0f, 0.0f};
  if (whole) w = *reinterpret_cast<f32x4 __attribute__((address_space(1)))*>(v);
  if (mine) zbar_quad((mt.nnz_base >> 2) + (uint64_t)tq, seed, step, z);
  double g;
  if constexpr (REDUCE) {
    __shared__ double scratch[2][16];
    double loss[2];
    block_sums_as_1024(a.partials, a.partials_per_sign, scratch, loss);
    g = (a.eps == 0.0f) ? 0.0 : (loss[0] - loss[1]) / (2.0 * (double)a.eps);
    if (blockIdx.x == 0 && threadIdx.x == 0) { a.scalars[0] = loss[0]; a.scalars[1] = loss[1]; a.scalars[2] = g; }
    if (!mine) return;
  } else {
    g = a.scalars[2];
  }
  const float c = (float)((double)a.lr * g);                          // lr * g, rounded once
  if (whole) {
    w[0] = fmaf(-c, z[0], w[0]); w[1] = fmaf(-c, z[1], w[1]); w[2] = fmaf(-c, z[2], w[2]); w[3] = fmaf(-c, z[3], w[3]);
    *reinterpret_cast<f32x4 __attribute__((address_space(1)))*>(v) = w;
  } else {
    for (int i = 0; j0 + i < (int64_t)mt.nnz; ++i) v[i] = fmaf(-c, z[i], v[i]);
  }
}

// ---- host side -----------------------------------------------------------------------------

static size_t small_lds_bytes(int r) {
  return (size_t)2 * SM_ROWS * r * SM_XSTRIDE * 2 + (size_t)3 * 4 * SM_CAP * 2;
}

static int64_t bands_of(const szo_linear_desc* d) { return (d->N + 63) / 64; }
static int64_t strips_of(const szo_linear_desc* d) { return (d->N + SM_BN - 1) / SM_BN; }

// What one launch consists of, as the rules below need it: sums over its matrices, K in units of 1024, entries in
// thousands.  A slice is 16 token rows.
struct LaunchShape {
  int64_t strips16 = 0, bands16 = 0;                        // 256-column strips and 64-row bands, times slices
  double band_k = 0.0, longest_k = 0.0;                     // K summed over those bands, longest K
  double slice_entries = 0.0, row_entries = 0.0;            // sensitive entries times slices, times token rows / 16
  double entries = 0.0, weights = 0.0, sum_k = 0.0;
  int64_t matrices = 0, tiles128 = 0, most_tokens = 0;      // 128 x 128 output tiles
  double tile_k = 0.0;                                      // K summed over those tiles
  bool bf16 = false;                                        // tile type of a layer
  void add(const szo_linear_desc* d) {
    if (d->M <= 0 || d->N <= 0) return;
    const int64_t slices = (d->M + SM_ROWS - 1) / SM_ROWS, tiles = ((d->M + 127) / 128) * ((d->N + 127) / 128);
    const double k = (double)d->K / 1024.0, nnz = (double)d->nnz * 1e-3;
    strips16 += strips_of(d) * slices;
    bands16 += bands_of(d) * slices;
    band_k += (double)(bands_of(d) * slices) * k;
    longest_k = std::max(longest_k, k);
    slice_entries += nnz * (double)slices;
    row_entries += nnz * (double)d->M / SM_ROWS;
    entries += nnz;
    weights += (double)d->N * (double)d->K;
    sum_k += k;
    ++matrices;
    most_tokens = std::max<int64_t>(most_tokens, d->M);
    tiles128 += tiles;
    bf16 = bf16 || d->tile_dtype == SZO_TILE_BF16;
    tile_k += (double)tiles * k;
  }
  double percent() const { return weights > 0.0 ? 1e5 * entries / weights : 0.0; }      // sensitive weights, in percent
};

// The stream kernel (small_m_kernel) needs whole 128-column blocks, the fp16 tile and 32-bit code offsets; the split
// kernel also takes the other uniform layers.
static bool stream_ok(const szo_linear_desc* d) {
  return d->K % 128 == 0 && d->tile_dtype == SZO_TILE_F16 && (uint64_t)(bands_of(d) * 64) * (uint64_t)d->K / 2 < (1ull << 32);
}

// Blocks of 16 token rows per pass of the stream kernel for a matrix of a launch.  Two (half as many passes over
// the weights) only pay when the launch is large: two-block workgroups run two to a CU instead of three, and a
// launch that fits the chip in one go is faster as more, smaller passes side by side.
constexpr int64_t kSmallWideWorkgroups = 1536;              // two rounds of the 768 workgroups the chip holds
static int g_force_rblocks = 0;                             // testing hook: 2 or 3 = that many wherever M > 16
void small_m_force_rblocks(int r) { g_force_rblocks = r; }
static int g_force_split = 0;                               // testing hook: 1 = always the split kernel, -1 = only where nothing else can
void small_m_force_split(int how) { g_force_split = how; }
static int small_m_rblocks(const szo_linear_desc* d, int64_t launch_wgs16) {
  if (d->M <= SM_ROWS) return 1;
  if (g_force_rblocks) return g_force_rblocks;
  if (launch_wgs16 <= kSmallWideWorkgroups) return 1;
  // fewest passes weighted by what a pass costs (measured on a 32-block 7B stack: 0.62, 0.79, 1.0 ms)
  const int64_t cost[3] = {62 * ((d->M + 15) / 16), 79 * ((d->M + 31) / 32), 100 * ((d->M + 47) / 48)};
  int best = 0;
  for (int r = 1; r < 3; ++r) if (cost[r] < cost[best]) best = r;
  return best + 1;
}

// Which kernel and instantiation a matrix of a launch runs with: a variant (stream kernel with 1, 2 or 3 blocks of
// token rows or with two activation sets; split kernel with one or two sets) and a dequantisation (uniform format
// with a group of 128; table format; other uniform groups; uniform layers whose other kernel is the tiled one, with
// either tile type).  Their number orders the step's table and launches.
enum { V_STREAM1, V_STREAM2, V_STREAM3, V_STREAM_DUAL, V_SPLIT, V_SPLIT_DUAL, kVariants };
enum { D_FAST, D_LUT, D_PLAIN, D_TILE_F16, D_TILE_BF16, kDequants };
constexpr int kClasses = kVariants * kDequants;
struct FewPlan {
  int variant, dequant;
  int part_shift = 0;                                       // split kernel: workgroups per band, see split_part_shift
  int cls() const { return variant * kDequants + dequant; }
  static FewPlan of_class(int cls) { return FewPlan{cls / kDequants, cls % kDequants, 0}; }
  bool split() const { return variant >= V_SPLIT; }
  bool dual() const { return variant == V_STREAM_DUAL || variant == V_SPLIT_DUAL; }
  int rblocks() const { return variant <= V_STREAM3 ? variant + 1 : variant == V_STREAM_DUAL ? 2 : 1; }
  int mode() const { return dequant == D_FAST ? SM_FAST : dequant == D_LUT ? SM_LUT : SM_PLAIN; }
  int rows() const { return dual() || split() ? SM_ROWS : SM_ROWS * rblocks(); }       // token rows of one slice
  int64_t units(const szo_linear_desc* d) const { return split() ? bands_of(d) << part_shift : strips_of(d); }   // workgroups per slice
  int slices(const szo_linear_desc* d) const { return (int)((d->M + rows() - 1) / rows()); }
};

// Whether a launch takes the split kernel.  The stream kernel's time is the chain of its longest K, which the split
// shortens, plus its share of the work; the split kernel pays for the sums of every band.  A mask of more than 0.1 % adds to
// both: the split kernel fetches the columns of x of every sensitive entry from memory, for every token row, where the
// stream kernel reads them from the staged x, one after the other along its chain.  Fitted to steps over single layers of
// 512..16384 rows x 512..16384 columns and one to four blocks, 1..448 tokens, 0.01..1 %, spread evenly and half in 1 % of the
// rows: the choice costs 0.2..0.7 % on average, and is up to 20 % slower than the stream kernel in 9 of 1948 cases (16384 x 4096
// at 40 tokens and 1 %: its last slice is half empty), where the rule without the mask was up to 33 % slower in 48.
// us per step, split against stream: 16384 x 2048 at 16 / 64 / 128 tokens 18 / 34 / 52 against 26 / 27 / 34; one / two / four
// OPT blocks at 16 tokens 47 / 66 / 125 against 130 / 134 / 158; one Llama block at 64 tokens and 0.01 / 0.1 / 0.4 / 1 %
// 76 / 89 / 155 / 297 against 90 / 98 / 142 / 223; four Mistral blocks at 1 % at 1 / 16 tokens 222 / 393 against 308 / 326.
// With groups of 32 and 64 the stream kernel loads its scales where it needs them; look-ups (table format) and two activation
// sets cost more per unit in the split kernel: three Llama blocks at 16 tokens with tables 165 against 145, one Mistral block
// with two sets at 16 / 32 tokens 70 / 116 against 134 / 139.
struct FewEstimate { double split, stream; };
static FewEstimate few_estimate(const LaunchShape& launch, bool dual, bool lut, bool plain) {
  const double percent = launch.percent(), over = std::max(percent - 0.1, 0.0), share = percent > 0.0 ? over / percent : 0.0;
  const double split = (lut ? 0.018 : 0.012) * (dual ? 1.65 : 1.0) * (double)launch.bands16 +
                       (lut ? 0.0068 : 0.0058) * (dual ? 1.65 : 1.0) * launch.band_k +
                       (0.012 * launch.row_entries + 0.008 * launch.slice_entries) * share * (dual ? 2.0 : 1.0);
  const double stream = ((plain ? 12.9 : 6.9) + 8.0 * over) * launch.longest_k + 0.0026 * launch.band_k;
  return FewEstimate{split, stream};
}
static bool split_pays(const LaunchShape& launch, bool dual, bool lut, bool plain) {
  const FewEstimate e = few_estimate(launch, dual, lut, plain);
  return e.split <= e.stream;
}
// Workgroups per band of a split launch, 1 << the result.  A band's wave dequantises four 16-row subtiles for each 128 columns, one
// after the other, which is most of a small launch's time: cut into two or four workgroups the band takes more CUs.  Each of them
// stages x and looks through the band's entries again, so only while all workgroups still have a CU to themselves (one
// forward at 16 tokens, us with 1 / 2 / 4 workgroups per band: 4096 x 4096 (64 bands) 10.4 / 7.7 / 6.6, 8192 x 4096 10.5 / 8.0 / 9.5,
// 11008 x 4096 10.8 / 11.3 / 12.7, 4096 x 16384 26.8 / 19.6 / 16.5); and in two where the chain of a long K outlasts the
// whole launch's work, both estimated as in split_pays, and its bands are a quarter of it at most (a step over one OPT block at
// 1 / 16 tokens, fc2's bands cut in two: 33.8 / 42.4 -> 31.1 / 35.5; where the chain is shorter it loses: one Mistral block 31.9 / 39.9 ->
// 36.2 / 41.8; so does a layer by itself: 1024 x 16384 at 200 tokens with groups of 32 32.3 -> 41.8).
static int split_part_shift(const szo_linear_desc* d, const LaunchShape& launch) {
  if (launch.bands16 <= 64) return 2;
  if (launch.bands16 <= 128) return 1;
  const double k = (double)d->K / 1024.0, chain = 3.2 + 1.55 * k, work = 0.012 * (double)launch.bands16 + 0.0058 * launch.band_k;
  return k >= 8.0 && 4 * bands_of(d) * ((d->M + SM_ROWS - 1) / SM_ROWS) <= launch.bands16 && chain > 1.1 * work ? 1 : 0;
}
static FewPlan few_plan(const szo_linear_desc* d, const LaunchShape& launch, bool dual, Partials less = kBandsInParts) {
  FewPlan p;
  if (d->format == SZO_FORMAT_LUT) p.dequant = D_LUT;
  else if (d->tile_dtype == SZO_TILE_BF16) p.dequant = D_TILE_BF16;
  else if (!stream_ok(d)) p.dequant = D_TILE_F16;
  else p.dequant = d->group == 128 ? D_FAST : D_PLAIN;
  bool split = split_pays(launch, dual, p.dequant == D_LUT, p.dequant == D_PLAIN);
  if (g_force_split) split = g_force_split > 0;
  if (g_force_rblocks || less == kStreamKernel) split = false;
  if (!stream_ok(d)) split = true;
  if (split) {
    p.variant = dual ? V_SPLIT_DUAL : V_SPLIT;
    p.part_shift = less == kBandsInParts ? split_part_shift(d, launch) : 0;
  }
  else p.variant = dual ? V_STREAM_DUAL : V_STREAM1 + small_m_rblocks(d, launch.strips16) - 1;
  return p;
}

// Codes of a matrix in bytes.
static int64_t code_bytes(const szo_linear_desc* d) { return (int64_t)((d->N + 63) / 64 * 64) * (d->K / 2); }

struct LaunchTotals {                                       // over a launch's matrices
  int slices = 0, subs = 1;                                 // most slices; most 16-row subtiles of a split workgroup
  int64_t units = 0, k = 0, rows = 0, code_bytes = 0;       // workgroups per slice, longest K, most token rows, codes
  int64_t live = 0;                                         // workgroups that have rows, their K in all
  double live_k = 0.0, entries = 0.0, weights = 0.0;
  void add(const FewPlan& p, const szo_linear_desc* d) {
    slices = std::max(slices, p.slices(d));
    subs = std::max(subs, 4 >> p.part_shift);
    units += p.units(d);
    live += p.units(d) * p.slices(d);
    live_k += (double)(p.units(d) * p.slices(d)) * (double)d->K;
    k = std::max(k, d->K);
    rows = std::max(rows, d->M);
    code_bytes += ::szo::code_bytes(d);
    entries += (double)d->nnz;
    weights += (double)d->N * (double)d->K;
  }
};
// Waves of a split workgroup.  Four, because the sum over the waves and the loss are spread over them; eight where
// each of them still has two subtiles of a 128-column block to itself; 16 for the longest K while every workgroup has a CU to itself.
// One forward at 16 tokens, us with 4 / 8 / 16 waves: 512 x 512 4.2 / 4.5 / 5.6 (bands in four parts, as all of these but the last two), 2048 x 1024
// 4.7 / 4.9 / 6.0, 4096 x 2048 5.7 / 5.5 / 7.1, 4096 x 4096 7.6 / 6.6 / 7.8, 4096 x 11008 16.2 / 12.2 / 11.9, 4096 x 16384
// 26.1 / 18.8 / 16.5, 8192 x 8192 17.8 / 12.9 / 13.1, 16384 x 4096 13.6 / 11.8 / 12.1.  With more workgroups than the chip holds at
// once the depth of the split matters less than what a workgroup costs.  us per step with 4 / 8 waves: one Llama block at 16 / 24 /
// 48 tokens (664 / 1328 / 1992 workgroups) 43.5 / 36.3, 55.1 / 57.1, 70.5 / 77.3, one OPT block at 64 tokens (2304) 83 / 93; with the
// sensitive weights rounded as in the tile for both signs, where the registers of eight waves leave no room for a second
// workgroup on a CU, a 5000 x 4160 layer at 48 / 77 tokens (237 / 395) 23.5 / 22.1, 30.8 / 35.3, a Llama block at 48 tokens 89 / 130.
// Sensitive entries are a chain of their own, a memory round trip per sixteen of them, which more waves shorten: sixteen waves
// where each would still have about 80 of a band's, in up to four slices; eight up to 2304 workgroups where a band of the longest K
// has many against the number of workgroups.  us with 8 / 16 waves: a forward at one token and 1 %, 11008 x 4096 17.8 / 15.8, 16384 x
// 4096 with half the entries in 1 % of the rows 42.2 / 35.4; below the line a step of 16384 x 8192 at 16 tokens and 0.1 % 28.0 / 29.0, with more slices
// one of 70 x 5120 at 1722 and 0.7 % 36.1 / 39.3.  us per step with 4 / 8 (e = entries of a band over workgroups; "rows": half of them in
// 1 % of the rows): two OPT blocks at one token, 0.05 %, rows (e = 0.46) 63 / 54, two Mistral blocks at 16 tokens, 0.1 %, rows (0.7)
// 92 / 74, three at one token, 0.3 %, rows (1.4) 152 / 129; below it three Llama blocks at 4 tokens and 0.05 % (0.2) 76 / 80.  Evenly spread
// entries gain nothing up to e = 2 or so (two OPT blocks at 32 tokens and 0.1 % 100 / 111), but nothing here tells the two apart.
// Where the accumulators take more registers: tables (two Llama blocks at 2 tokens and 0.2 % (1) 86 / 107), and v and eps z rounded
// together for both signs: one Llama block with the bf16 tile at 16 tokens and 0.5 % (5.3) 89 / 79, at 4 and 0.2 % (2.1) 51 / 52; where all
// K are about the longest and its chain is hidden, as in slices of one layer, 5000 x 4160 at 160 tokens and 1 % (3.4) 115 / 130, 1770 x
// 15680 at 228 and 1 %, rows (24) 253 / 294; more workgroups, two OPT blocks at 21, 0.2 %, rows (0.9) 141 / 197, at one
// token and 0.5 % (4.6) 95 / 114, one at 32, 1 %, rows (9) 338 / 248.  Between those lines rows full of entries take up to 8 % longer
// with four than with eight, 11 % with tables, evenly spread ones 17 to 40 % less (two Llama blocks with tables at 4 tokens and 1 % (5.3),
// rows 252 / 228, evenly spread 157 / 190).
static int split_waves(const FewPlan& p, bool one_sign, int64_t workgroups, const LaunchTotals& t) {
  const int64_t blocks = (t.k + 127) / 128;
  const double band_entries = 64.0 * (double)t.k * t.entries / t.weights;      // of a band of the longest K, on average
  const bool both_rounded = p.dequant >= D_TILE_F16 && !one_sign, one_k = 2.0 * (double)t.k * (double)t.live < 3.0 * t.live_k;
  const double many = both_rounded && one_k ? 1e30 : !both_rounded && p.dequant != D_LUT ? 0.45 : workgroups <= 1024 ? 2.5 : 6.0;
  const int64_t wide = p.dual() || band_entries > many * (double)workgroups ? 2304 : both_rounded ? 256 : 1024;
  if (workgroups > wide || blocks * t.subs < 16) return 4;
  return workgroups <= 256 && (blocks > 96 || (t.slices <= 4 && 0.25 * t.subs * band_entries >= 1300.0)) ? 16 : 8;
}

template <int MODE, int R, bool DUAL>
static void launch_variant(dim3 blocks, const SmallArgs& a, hipStream_t stream) {
  const size_t lds = small_lds_bytes(R);
  if (a.stream_once) small_m_kernel<MODE, R, DUAL, true><<<blocks, 256, lds, stream>>>(a);
  else small_m_kernel<MODE, R, DUAL, false><<<blocks, 256, lds, stream>>>(a);
}
template <int R, bool DUAL>
static void launch_mode(int mode, dim3 blocks, const SmallArgs& a, hipStream_t stream) {
  if (mode == SM_FAST) launch_variant<SM_FAST, R, DUAL>(blocks, a, stream);
  else if (mode == SM_LUT) launch_variant<SM_LUT, R, DUAL>(blocks, a, stream);
  else launch_variant<SM_PLAIN, R, DUAL>(blocks, a, stream);
}
// The rule for the non-temporal stream of codes: one slice per strip and more codes in
// the launch than the 256 MB last-level (memory-side) cache of the chip keeps from one step to the next.
constexpr int64_t kLastLevelCacheBytes = 256ll << 20;
static bool g_force_stream_once = false;                    // testing hook: the stream for every one-slice launch
void small_m_force_stream_once(bool on) { g_force_stream_once = on; }
static int stream_once_rule(int slices, int64_t launch_code_bytes) {
  return slices == 1 && (g_force_stream_once || launch_code_bytes > kLastLevelCacheBytes);
}

// One launch of the matrices described by `a` (their table or the single one).
static int launch_plan(const FewPlan& p, const LaunchTotals& t, bool one_sign, SmallArgs& a, hipStream_t stream) {
  if (t.units * t.slices > 0x7FFFFFFF) return SZO_EUNSUPPORTED;
  a.slices = t.slices;
  a.few_rows = t.rows <= 4;
  a.stream_once = stream_once_rule(t.slices, t.code_bytes);
  const int wgs = (int)(t.units * t.slices);
  int rc = timing_begin(stream);
  if (rc != SZO_OK) return rc;
  if (p.split()) {
    rc = split_launch(SplitLaunch{p.mode(), p.dual(), p.dequant == D_TILE_BF16, p.dequant >= D_TILE_F16, one_sign, t.subs,
                                  split_waves(p, one_sign, wgs, t), wgs, t.k}, a, stream);
    if (rc != SZO_OK) return rc;
  } else {
    const dim3 blocks((unsigned)wgs);
    if (p.dual()) launch_mode<2, true>(p.mode(), blocks, a, stream);
    else if (p.rblocks() == 1) launch_mode<1, false>(p.mode(), blocks, a, stream);
    else if (p.rblocks() == 2) launch_mode<2, false>(p.mode(), blocks, a, stream);
    else launch_mode<3, false>(p.mode(), blocks, a, stream);
    SZO_LAUNCH_CHECK();
  }
  return timing_end(stream);
}

// The step also takes matrices with more tokens: they run as slices of 16 or 32 token rows, each a pass
// of its own over the weights.  On a 32-block 7B-shaped stack a 32-row pass takes 0.8-0.9 ms and a row of
// 256x256 tiles of the tiled kernel 6.4 ms, whatever part of its 256 rows is padding: slicing wins while
// ceil(M/32) stays below 7.5 ceil(M/256), e.g. up to 224 tokens and from 257 to 448; beyond 15 such
// slices the tiled kernel is the default (SZO_STEP_ONE_DENSE_PASS overrides that).
constexpr int kSmallMaxSlices = 15;
// Uniform layers that only the split kernel takes (bf16 tile, K an odd multiple of 64), against 128x128 tiles.  Measured with
// the bf16 tile, us per step: one Llama block at 16 / 64 / 128 tokens 62 / 134 / 302 against 371 / 375 / 379, sixteen blocks
// 788 / 2934 / 2477 against 3047 / 3106 / 3204.  From 65 tokens on only where the tiles would leave the chip idle (2304 workgroups here).
constexpr int64_t kSplitOnlyTokens = 64, kSplitOnlyTwoSets = 1536;
// Inside these limits both are estimated: the split kernel by its bands and their entries or the chain of the longest K, the
// tiles by the chain of the longest K or their share of the work, one launch after the other where they are too few for a
// grouped one.  Fitted, in about us, to steps and single-layer losses with the bf16 tile over the same shapes, masks spread
// evenly and half in 1 % of the rows: 20 of 3028 cases are more than 3 % slower than the tiles (20 % at most: a 300 x 320 layer at
// one token), where token counts alone left 74 (65 %).  us per step at 1 %, split against tiles: a 16384 x 4096 layer at 64 / 128
// tokens 140 / 266 against 191 / 186, three Llama blocks at 64 tokens 869 against 689, one OPT block at 128 tokens 437 against 463.
// Beyond 128 tokens (single layers of 64..16384 rows x 256..16384 columns at 129..4000, 0.01..1 %) a band's time goes with its columns and
// entries, those of a second set of activations on top, which is measured up to 1536 bands and slices (kSplitOnlyTwoSets), and a
// tile's walk takes longer, more so with the bf16 tile and with two launches for a step.  us on the split kernel against the others:
// 4059 x 6848 at 473 tokens and 0.3 % 154 against 141 on the one-dense-pass kernel, a forward of 810 x 9280 at 2238 185 against 133 in tiles;
// two sets of 4096 x 4160 at 200 and 1 % 204 against 185, of 2354 x 704 at 953 (2220 bands and slices) 72 against 51, of
// 3552 x 12416 at 329 248 against 378.
// (All of these are tiles with K whole.  With K in two parts, which the estimates leave out, a few sizes near the line are 5..20 % faster
// in tiles: 4096 x 4096 at 128 tokens and 1 % with the bf16 tile.)
static double split_rounded_us(const LaunchShape& l, bool two_sets) {
  const double chain = l.longest_k * (1.9 + 5.3 * l.percent());
  if (l.most_tokens <= 128) return 13.5 + std::max(0.016 * (double)l.bands16 + 0.0036 * l.band_k + 0.02 * l.slice_entries, chain);
  const double columns = 0.005 * (double)l.bands16 + 0.0062 * l.band_k;
  return 13.5 + (two_sets ? std::max(1.65 * columns + 0.06 * l.slice_entries, 1.65 * chain) : std::max(columns + 0.03 * l.slice_entries, chain));
}
static double tiled_us(const LaunchShape& l, int forwards) {
  const double chain = (l.most_tokens <= 128 ? 9.1 : (forwards == 1 ? 11.5 : 12.5) + (l.bf16 ? 2.0 : 0.0)) * (1.0 + 0.05 * l.percent()), share = 0.0123 * forwards * l.tile_k * (1.0 + 0.73 * l.percent());
  const bool one_launch = l.matrices == 1 ? forwards == 1 : forwards * l.tiles128 >= 384;
  return 7.0 + 11.3 * (double)(forwards * l.matrices) + std::max(chain * (one_launch ? l.longest_k : forwards * l.sum_k), share);
}
// The split kernel's byte offsets inside a band's codes (32 per column) and inside its sixteen rows of x (32 per column)
// have 32 bits; stream_ok's bound on the codes keeps the other layers below that.
constexpr int64_t kSplitOnlyColumns = 1 << 23;
// Whatever the number of tokens: launches that end before the other kernels have walked the longest K, which take at least the
// time below for it however little work there is (their tiles are then few, and each has all of K to itself).  Measured, us,
// other kernels -> this path: a forward of a 300 x 4096 layer at 450 / 1000 / 4000 tokens 55 / 56 / 56 -> 11 / 17 / 46, 64 x 16384 at
// 600 / 8000 tokens 203 / 208 -> 21 / 80, 1024 x 4096 at 600 / 2000 tokens 56 / 57 -> 26 / 48, 4096 x 1024 at 450 tokens 18.9 -> 15.4;
// steps of the same 132 / 69 / 78 -> 18 / 25 / 50, 422 / 208 -> 28 / 88, 65 / 66 -> 35 / 57, 29.7 -> 23.8; beyond the line a step over 4096 x
// 4096 at 600 tokens 67 -> 68, a forward 57 -> 59, of 258 x 5248 at 6437 69 -> 78.  Forwards with tables (256 x 256 tiles): 300 x 4096 at
// 6000 tokens 87 -> 102, 445 x 9984 at 3681 232 -> 176, 4096 x 4096 at 450 87 -> 78, 1231 x 15872 at 1741 353 -> 398.  The bf16 tile (and K an odd multiple of 64) compares its own estimates below: a
// forward of a 1024 x 1024 / 4096 x 4096 layer at 300 tokens 21 / 70 -> 9 / 45.
// (Below 1024 columns the chain is a few launches' time and either path's launches weigh more.  The tiles' times are of tiles that walk K as a
// whole, with a schedule that scattered behind its last matrix instruction; with K in two parts they take up to 40 % less.  The line stays
// for what moves with it beside the time: the tiles round v + eps z, and with groups of 128 the dequantised weights, which the few-token
// kernels do not.  Unperturbed forwards with small groups, where nothing of that differs, have a line of their own, two_part_tiles_win.)
static bool outruns_the_chain(const szo_linear_desc* d, const LaunchShape& launch, int forwards) {
  if (d->K < 1024) return false;
  const bool lut = d->format == SZO_FORMAT_LUT, plain = !lut && d->group != 128, single = forwards == 1;      // (a table layer's group means nothing)
  const FewEstimate e = few_estimate(launch, d->x_minus && !single, lut, plain);
  // (the estimates are of steps up to 448 tokens: with groups below 128 and dense masks a forward over more of them takes up to that much longer.)
  // A single forward has the others' time against it once, not twice: there the estimate has to hold.  The stream kernel computes
  // whole strips of 256 rows for every slice, with tables at the price of their look-ups (which the choice of the kernel leaves out); the
  // split kernel's time goes with columns and entries as in split_rounded_us below (692 x 15872 at 2253 tokens 201 in tiles, 236 there).
  const double strip_k = 4.0 * (double)launch.strips16 * launch.longest_k;
  const double stream = e.stream + (single ? (lut ? 0.00675 : 0.0026) * strip_k - 0.0026 * launch.band_k : 0.0) + 3.0 + 0.0015 * (double)launch.bands16;
  const double split = e.split * (plain ? 1.35 : 1.0), dense = 1.0 + 0.8 * std::max(launch.percent() - 0.1, 0.0);
  double few = dense * (!single ? std::min(split, stream) : e.split <= e.stream ? split : stream);
  if (single && !lut && e.split <= e.stream) few = std::max(few, 0.005 * (double)launch.bands16 + 0.0062 * launch.band_k + 0.03 * launch.slice_entries);
  return few < (!single ? 10.0 + 11.8 * launch.longest_k : 5.0 + (lut ? 20.0 : 12.7) * launch.longest_k);
}
// An unperturbed single forward of a layer with groups below 128 against 128 x 128 tiles that compute K in two parts
// (tiles_halve_k).  Without a perturbation the tiles round what these few-token launches round, the dequantised weights and v, and either error is the
// same.  Perturbed forwards stay: the few-token kernels round v and z one by one, the tiles v + eps z, which leaves 14 times the
// error in y(+) - y(-) (2.1e-4 -> 2.9e-3 of it with v ~ 0.02, eps = 1e-3).  Groups of 128 and tables stay: there the few-token kernels
// do not round the dequantised weights at all.
// The tiles take the chain of half of K whatever the number of tokens, 8 % more per 64 tiles beyond 128 and 10 % more at 1 %.
// The few-token estimates are as above, the split kernel's at its lower side (0.8..1.2 of it, with dense masks a third more), so that a
// call moves where the tiles are faster by more than the estimate's spread.  us with 0.1 % / 1 % sensitive, few-token kernels -> tiles
// (in brackets: the tiles where the few-token kernels stay): 4096 x 4096 at 256 tokens 33 (34), at 440 52 -> 35; 11008 x 4096 at 64
// tokens 26 (30), at 128 43 -> 35; 10241 x 2944 at 269 56 -> 29; 5831 x 3200 at 196 33 -> 28; 3284 x 512 at 354 11.8 -> 9.6; 9359 x
// 512 at 69 9.0 (9.3); 6140 x 10752 at 189 - / 297 -> 96, 2034 x 1152 at 317 - / 30 -> 14, 13245 x 256 at 43 - / 9.4 -> 6.9.
// (256 columns in 193 to 256 tiles are computed whole, see tiles_halve_k.  The estimate, 9.4 at 1 %, holds for them too: 25000 rows at 43 / 100 /
// 128 tokens 11.6 / 15.4 / 18.0 -> 8.1 / 9.0 / 9.2, half the entries in 1 % of the rows 19.7 -> 10.4; 6300 at 440 15.5 -> 9.2.)
static bool two_part_tiles_win(const szo_linear_desc* d) {
  LaunchShape launch;
  launch.add(d);
  if (d->format != SZO_FORMAT_UNIFORM || d->group == 128 || !stream_ok(d) || launch.tiles128 > kTwoPartTiles || d->K < kTwoPartColumns) return false;
  if (g_force_split || g_force_rblocks || g_force_stream_once) return false;                 // testing hooks that name a few-token kernel
  const FewEstimate e = few_estimate(launch, false, false, true);
  const double few = (e.split <= e.stream ? 0.85 * e.split : e.stream + 2.0) * (1.0 + 0.35 * std::max(launch.percent() - 0.1, 0.0));
  const double wide = 1.0 + 0.17 * std::max((double)(launch.tiles128 - 128), 0.0) / 128.0;
  return (6.0 + 7.2 * launch.longest_k) * wide * (1.0 + 0.1 * launch.percent()) < few;
}
static bool layer_eligible(const szo_linear_desc* d, const LaunchShape& launch, int forwards) {
  if (!stream_ok(d))
    return d->format == SZO_FORMAT_UNIFORM && d->K < kSplitOnlyColumns &&
           (launch.bands16 <= 2304 || d->M <= kSplitOnlyTokens) &&
           (!(d->x_minus && forwards == 2) || d->M <= 128 || launch.bands16 <= kSplitOnlyTwoSets);
  if (outruns_the_chain(d, launch, forwards)) return true;
  // two activation sets: a pass holds 16 token rows of each, so it is worth less
  const int64_t slices = (d->M + (d->x_minus ? 15 : 31)) / (d->x_minus ? 16 : 32), tile_rows = (d->M + 255) / 256;
  return slices <= kSmallMaxSlices && 2 * slices < 15 * tile_rows;
}
// `separate`: every matrix is a launch of its own (then the sums of their times are compared).
static double rounded_us(const szo_linear_desc* descs, int n, bool split, int forwards, bool separate) {
  if (!separate) {
    LaunchShape shape;
    bool two_sets = false;
    for (int i = 0; i < n; ++i) {
      shape.add(&descs[i]);
      two_sets = two_sets || (forwards == 2 && descs[i].x_minus);
    }
    return split ? split_rounded_us(shape, two_sets) : tiled_us(shape, forwards);
  }
  double us = 0.0;
  for (int i = 0; i < n; ++i) us += rounded_us(&descs[i], 1, split, forwards, false);
  return us;
}
double small_m_rounded_us(const szo_linear_desc* descs, int n, bool few, bool separate) { return rounded_us(descs, n, few, 2, separate); }
bool small_m_eligible(const szo_linear_desc* descs, int n, bool any_token_count, bool separate, int forwards) {
  LaunchShape shape;
  for (int i = 0; i < n; ++i) shape.add(&descs[i]);
  bool all_stream = true;
  for (int i = 0; i < n; ++i) {
    const szo_linear_desc* d = &descs[i];
    if (d->M <= 0 || d->N <= 0) continue;                   // an empty layer contributes nothing on either path
    if (separate && forwards == 2 && d->x_minus) return false;
    if (!(any_token_count ? stream_ok(d) : layer_eligible(d, shape, forwards))) return false;
    all_stream = all_stream && stream_ok(d);
  }
  return n > 0 && (all_stream || rounded_us(descs, n, true, forwards, separate) <= rounded_us(descs, n, false, forwards, separate));
}
bool small_m_takes_forward(const szo_linear_desc* d, bool perturbed) {
  return small_m_eligible(d, 1, false, false, 1) && (perturbed || !two_part_tiles_win(d));
}
static FewPlan plan_of_one(const szo_linear_desc* d, Partials less) {
  LaunchShape shape;
  shape.add(d);
  return few_plan(d, shape, false, less);
}
int64_t small_m_launch_partials(const szo_linear_desc* d, Partials less) {
  const FewPlan p = plan_of_one(d, less);
  return p.units(d) * p.slices(d);
}

size_t small_m_table_bytes(int n) { return sizeof(SmallMat) * (size_t)n; }

static void fill_mat(SmallMat& m, const szo_linear_desc* d) {
  m.x = (const uint16_t*)d->x; m.x2 = (const uint16_t*)d->x_minus; m.qweight = d->qweight;
  m.scales = (const uint16_t*)(d->format == SZO_FORMAT_LUT ? d->lut : d->scales);
  m.tile_ptr = d->tile_ptr; m.sp_idx = d->sp_idx; m.sp_val = d->sp_val;
  m.target = (const uint16_t*)d->target; m.y = d->y;
  m.nnz_base = d->nnz_base;
  m.loss_scale = 1.0 / ((double)d->M * (double)d->N);
  m.N = (int)d->N; m.K = (int)d->K; m.M = (int)d->M; m.nnz = (uint32_t)d->nnz;
  int gs = 0;
  while (d->format == SZO_FORMAT_UNIFORM && (1 << gs) < d->group) ++gs;
  m.group_shift = gs;
  int l = 0;
  while ((1ull << l) < (uint64_t)m.K) ++l;
  m.div_mul = (uint32_t)((((1ull << l) - (uint64_t)m.K) << 32) / (uint64_t)m.K + 1ull);
  m.div_shift = l - 1;
  m.first_block = 0; m.partial_base = 0; m.first_quad = 0;
}

// Dynamic LDS limit of every instantiation, once per device.
template <int MODE, int R, bool DUAL>
static int set_attrs_of() {
  static std::atomic<uint64_t> done[2];
  int rc = set_lds_limit_once(done[0], (const void*)small_m_kernel<MODE, R, DUAL, false>, small_lds_bytes(R));
  if (rc != SZO_OK) return rc;
  return set_lds_limit_once(done[1], (const void*)small_m_kernel<MODE, R, DUAL, true>, small_lds_bytes(R));
}
template <int R, bool DUAL>
static int set_attrs_of_modes() {
  int rc = set_attrs_of<SM_FAST, R, DUAL>();
  if (rc == SZO_OK) rc = set_attrs_of<SM_PLAIN, R, DUAL>();
  if (rc == SZO_OK) rc = set_attrs_of<SM_LUT, R, DUAL>();
  return rc;
}
static int set_small_attrs() {
  static std::atomic<uint64_t> all_done{0};                   // one look instead of one per instantiation
  int dev = 0;
  SZO_HIP(hipGetDevice(&dev));
  if (all_done.load(std::memory_order_acquire) & (1ull << (dev & 63))) return SZO_OK;
  int rc = set_attrs_of_modes<1, false>();
  if (rc == SZO_OK) rc = set_attrs_of_modes<2, false>();
  if (rc == SZO_OK) rc = set_attrs_of_modes<3, false>();
  if (rc == SZO_OK) rc = set_attrs_of_modes<2, true>();
  if (rc == SZO_OK) all_done.fetch_or(1ull << (dev & 63), std::memory_order_release);
  return rc;
}

// One matrix, descriptor passed in the kernel arguments (no device table needed), as one launch.  In loss mode
// slice i writes its partials behind those of slice i - 1, small_m_launch_partials(d, less) in all, scaled by 1 / (M N) of the
// whole matrix, so that their sum is the matrix's loss.  store_sign: the forward whose outputs are written to d->y, 0 = none.
int small_m_launch_one(const szo_linear_desc* d, uint64_t seed, uint64_t step, float eps, int store_sign, bool loss_mode,
                       bool both_signs, double* partial_plus, double* partial_minus, Partials less, hipStream_t stream) {
  const int rc = set_small_attrs();
  if (rc != SZO_OK) return rc;
  const FewPlan p = plan_of_one(d, less);
  SmallArgs a{};
  fill_mat(a.inl[0], d);                                       // whole matrix: the kernel offsets rows by slice
  a.part_shifts = (uint32_t)p.part_shift;
  a.table = nullptr; a.n_mats = 1;
  a.store_sign = store_sign; a.loss_mode = loss_mode ? 1 : 0;
  a.seed = seed; a.step = step; a.eps = eps;
  if (!both_signs && store_sign < 0) { a.eps = -eps; a.store_sign = 1; }     // the wanted forward is the "+" one
  a.partial_plus = partial_plus;
  a.partial_minus = partial_minus;
  LaunchTotals t;
  t.add(p, d);
  return launch_plan(p, t, !both_signs, a, stream);
}

// When every workgroup of the update adds up the partials by itself instead of waiting for a launch that does: few partials,
// because their sum stands at the beginning of each workgroup's chain, and few workgroups, because each of them reads all.
// Single layers, us per step with a launch of its own -> here: 16 partials per sign and 1 workgroup 14.1 -> 13.8, 64 and 17
// 20.3 -> 20.1, 256 and 17 13.8 -> 13.6, 128 and 328 25.8 -> 25.4; beyond the line 400 and 2 16.9 -> 17.4, 1216 and 17
// 51.7 -> 52.2, 256 and 656 27.4 -> 28.1, one OPT block at 16 tokens (576 and 202) 41.7 -> 42.4.
constexpr int64_t kFusedReducePartials = 256, kFusedReduceWorkgroups = 256;

// A whole stack in one launch per instantiation.  The table is assembled on the host, longest K
// first (their workgroups run longest, so they should start first), and travels in the kernel arguments
// (up to kInlineMats matrices) or is copied into `table_dev` (device, small_m_table_bytes(n)) with an
// asynchronous copy on the stream; it also drives one grouped sparse update.  With `do_forward` false only the
// update runs (used by the other paths): `partials_per_sign` > 0 says that g has still to be formed from
// that many loss partials per sign.
int small_m_step(const szo_linear_desc* descs, int n, uint64_t seed, uint64_t step, float eps, float lr,
                 void* table_dev, double* partial_plus, int64_t partials_per_sign, double* scalars, bool do_forward,
                 hipStream_t stream) {
  int rc = do_forward ? set_small_attrs() : SZO_OK;
  if (rc != SZO_OK) return rc;
  if (n > kMaxStepMatrices || (n > kInlineMats && !table_dev)) return SZO_EUNSUPPORTED;
  LaunchShape shape;
  for (int i = 0; i < n; ++i) shape.add(&descs[i]);
  // two activation sets (forward launches only): one block of rows for each, whatever the token count
  auto plan_for = [&](const szo_linear_desc* d) {
    FewPlan p = few_plan(d, shape, do_forward && d->x_minus != nullptr);
    if (n > kInlineMats) p.part_shift = 0;                  // (part_shifts belongs to the table in the arguments)
    return p;
  };
  if (small_m_table_bytes(n) > kTableBytesPerMatrix * (size_t)kMaxStepMatrices) return SZO_EUNSUPPORTED;
  static thread_local std::vector<SmallMat> host_table;
  host_table.resize((size_t)std::max(n, 1));
  SmallMat* const host = host_table.data();
  // order: by instantiation, inside each by K descending
  static thread_local std::vector<std::pair<int64_t, int>> order;
  order.resize((size_t)n);
  for (int i = 0; i < n; ++i)
    order[(size_t)i] = {((int64_t)plan_for(&descs[i]).cls() << 40) - descs[i].K, i};
  std::sort(order.begin(), order.end());
  // One table entry per matrix; a launch has (units of its matrices) x (slices of its longest matrix)
  // workgroups (those past a matrix's last slice return at once), and slice i of a matrix writes its
  // loss partials behind those of slice i - 1.
  struct ClassTotals : LaunchTotals { int entries = 0; } classes[kClasses];
  int entries = 0;
  int64_t quads = 0, partials = 0;
  for (const auto& o : order) {
    const szo_linear_desc* d = &descs[o.second];
    const FewPlan p = plan_for(d);
    ClassTotals& c = classes[p.cls()];
    // a layer without tokens or outputs has no workgroups; it keeps its table entry for the update
    const bool live = d->M > 0 && d->N > 0;
    const int slices = live ? p.slices(d) : 0;
    const int64_t units = live ? p.units(d) : 0;
    SmallMat& m = host[entries++];
    fill_mat(m, d);
    m.first_block = (int)c.units;
    m.partial_base = (int)partials;
    m.first_quad = quads;
    if (live) c.add(p, d);
    ++c.entries;
    partials += units * slices;
    quads += (((int64_t)d->nnz + 3) / 4 + 63) & ~(int64_t)63;      // a wave of the update serves one matrix
    if (do_forward && 2 * partials > kMaxLossPartials) return SZO_EUNSUPPORTED;
    if (c.units * c.slices > 0x7FFFFFFF) return SZO_EUNSUPPORTED;
  }
  const bool inl = entries <= kInlineMats;
  if (!inl) {
    rc = stage_table(host, sizeof(SmallMat) * (size_t)entries, table_dev, stream);
    if (rc != SZO_OK) return rc;
  }
  const SmallMat* tdev = inl ? nullptr : (const SmallMat*)table_dev;
  if (do_forward) {
    SmallArgs a{};
    a.store_sign = 0; a.loss_mode = 1;
    a.seed = seed; a.step = step; a.eps = eps;
    a.partial_plus = partial_plus; a.partial_minus = partial_plus + partials;
    int first_entry = 0;
    for (int cls = 0; cls < kClasses; ++cls) {
      const ClassTotals& c = classes[cls];
      if (c.units > 0 && c.slices > 0) {
        a.table = inl ? nullptr : tdev + first_entry;
        a.part_shifts = 0;
        if (inl) std::copy(host + first_entry, host + first_entry + c.entries, a.inl);
        for (int e = 0; inl && e < c.entries; ++e) a.part_shifts |= (uint32_t)plan_for(&descs[order[(size_t)(first_entry + e)].second]).part_shift << (4 * e);
        a.n_mats = c.entries;
        rc = launch_plan(FewPlan::of_class(cls), c, false, a, stream);
        if (rc != SZO_OK) return rc;
      }
      first_entry += c.entries;
    }
    partials_per_sign = partials;
  }
  const int64_t ub = (quads + 255) / 256;
  if (ub > 0x7FFFFFFF) return SZO_EUNSUPPORTED;
  const bool reduce_here = ub > 0 && ub <= kFusedReduceWorkgroups && partials_per_sign > 0 && partials_per_sign <= kFusedReducePartials;
  // (a step without a single live layer has no partials: its losses are the sums over none)
  if (!reduce_here && (do_forward || partials_per_sign > 0)) {
    rc = reduce_step(partial_plus, (int)partials_per_sign, eps, scalars, stream);
    if (rc != SZO_OK) return rc;
  }
  if (ub > 0) {
    InlineUpdateArgs with_table{};
    UpdateArgs& u = with_table.staged;
    u.table = tdev;
    if (inl) std::copy(host, host + entries, with_table.inl);
    u.n_mats = entries; u.total_quads = quads;
    u.partials_per_sign = reduce_here ? (int)partials_per_sign : 0;
    u.partials = partial_plus; u.scalars = scalars;
    u.seed = seed; u.step = step; u.lr = lr; u.eps = eps;
    if ((rc = timing_begin(stream, 1)) != SZO_OK) return rc;
    if (inl && reduce_here) sparse_update_table_kernel<true><<<(unsigned)ub, 256, 0, stream>>>(with_table);
    else if (inl) sparse_update_table_kernel<false><<<(unsigned)ub, 256, 0, stream>>>(with_table);
    else if (reduce_here) sparse_update_table_kernel<true><<<(unsigned)ub, 256, 0, stream>>>(u);
    else sparse_update_table_kernel<false><<<(unsigned)ub, 256, 0, stream>>>(u);
    SZO_LAUNCH_CHECK();
    if ((rc = timing_end(stream)) != SZO_OK) return rc;
  }
  return SZO_OK;
}

}  // namespace szo
