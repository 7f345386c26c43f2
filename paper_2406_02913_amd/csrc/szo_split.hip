// Few-token kernel for launches that do not fill the chip: K split over the waves of a workgroup.
//
// A launch over one layer or one decoder block has too few 256-column strips to occupy 256 CUs, and what it then
// waits for is not bandwidth but the serial walk of a wave along K: one 4096 x 4096 layer at one token has 64 bands
// of 64 rows, i.e. 64 waves on a chip that holds 4096, each of which takes 31 us for its 32 blocks of 128 columns
// (120 us at K = 16384).  Here a workgroup is ONE band and one slice of 16 token rows, and its 2..16 waves take
// consecutive parts of K.  Nothing is shared inside the loop -- a wave reads its own columns of x straight into
// registers, there is no staging and no barrier -- and the waves' accumulators are added through LDS, in wave order,
// before the epilogue.  More splits mean shorter chains; the whole sum stays inside one workgroup, so no second
// kernel and no partial outputs in memory are needed.
//
// Where that leaves CUs idle, a band is cut further, into two or four workgroups of 32 or 16 rows (part_shifts, chosen by
// split_part_shift): each stages x again and looks through the band's entries again, but dequantises only its own rows.
//
// The arithmetic is that of small_m_kernel: y(+-) = x dq^T + x v^T +- eps x z^T, un-centred codes with the block's
// scale applied in fp32 for groups of 128, the sensitive entries as one-hot matrix products of 16 entries.
// With several slices each of them reads the band's codes (neighbouring workgroups of one XCD, through its L2).
//
// Measured, us of GPU time per call in a graph, with whole bands and 16 waves -> cut bands, x staged for the token rows that
// exist and two entries per lane: a 4096 x 4096 forward at 1 / 16 tokens 9.8 / 11.6 -> 5.3 / 6.6, 4096 x 16384 21.8 / 27.5 ->
// 11.2 / 16.8, 16384 x 4096 (bands whole) 11.0 / 13.1 -> 9.5 / 11.8.  An empty launch takes 3.4 there; the rest is a chain of a few
// memory round trips (table, tile bounds, entries, their columns of x) beside the dequantisation.  Against the stream
// kernel: a step over one OPT block at 1 / 16 tokens 128 / 130 -> 31 / 36, a Llama block with the bf16 tile at 16 tokens,
// which the tiled kernel ran before, 371 -> 62; from ~3000 workgroups on the x and the sums of every band cost more than
// the stream kernel's idle waves.
#include <atomic>
#include <type_traits>
#include "szo_few.h"
#include "szo_nonfinite.h"

namespace szo {

typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef short short4_t __attribute__((ext_vector_type(4)));
typedef float float2_t __attribute__((ext_vector_type(2)));

constexpr int SP_WIN = 128;             // sensitive entries computed per refill of a wave's window, two per lane
constexpr int SP_WIN_FLOATS = SP_WIN * 10 / 4;             // of a window: column, row, two 16-bit values
constexpr int SP_MAX_WAVES = 16;
constexpr int SP_XROW = 128 + 8;        // LDS row stride of a staged block of x, in 16-bit elements

// Operand types and the two matrix products per 16-bit tile type.  fp16: operands in the element order
// (0,4)(1,5)(2,6)(3,7), see sm_dequant_word; bf16: in natural order, activations unchanged.
template <bool BF16> struct SplitOps;
template <> struct SplitOps<false> {
  typedef half8_t frag;
  static __device__ __forceinline__ frag activations(u32x4 u) {
    const u32x4 w = {sm_stage_x_word(u, 0), sm_stage_x_word(u, 1), sm_stage_x_word(u, 2), sm_stage_x_word(u, 3)};
    return __builtin_bit_cast(half8_t, w);
  }
  static __device__ __forceinline__ uint16_t narrow(float v) { return __builtin_bit_cast(uint16_t, (_Float16)v); }
  static __device__ __forceinline__ uint16_t activation(uint16_t bits) {      // same truncation as the staged form
    auto h = __builtin_amdgcn_cvt_pkrtz(__uint_as_float((uint32_t)bits << 16), 0.0f);
    return (uint16_t)(__builtin_bit_cast(uint32_t, h) & 0xFFFFu);
  }
  static __device__ __forceinline__ float4_t dense(frag x, frag w, float4_t c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_f16(x, w, c, 0, 0, 0);
  }
  static __device__ __forceinline__ float4_t sparse(u32x2 x, u32x2 w, float4_t c) {
    return __builtin_amdgcn_mfma_f32_16x16x16f16(__builtin_bit_cast(half4_t, x), __builtin_bit_cast(half4_t, w), c, 0, 0, 0);
  }
};
template <> struct SplitOps<true> {
  typedef bf16x8_t frag;
  static __device__ __forceinline__ frag activations(u32x4 u) { return __builtin_bit_cast(bf16x8_t, u); }
  static __device__ __forceinline__ uint16_t narrow(float v) { return __builtin_bit_cast(uint16_t, (__bf16)v); }
  static __device__ __forceinline__ uint16_t activation(uint16_t bits) { return bits; }
  static __device__ __forceinline__ float4_t dense(frag x, frag w, float4_t c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(x, w, c, 0, 0, 0);
  }
  static __device__ __forceinline__ float4_t sparse(u32x2 x, u32x2 w, float4_t c) {
    return __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(__builtin_bit_cast(short4_t, x), __builtin_bit_cast(short4_t, w), c, 0, 0, 0);
  }
};

// Eight codes -> eight bf16 weights (c - 8) s in natural order, each rounded once.  Two nibbles at a time become 1024 + c and
// 64 + c in fp16 (as in sm_dequant_word); a mixed-precision fma takes them to (c - 8) s, exact in fp32: 17 instructions, where
// extracting and converting every code by itself took 28.
__device__ __forceinline__ bf16x8_t dequant_word_bf16(uint32_t q, _Float16 s) {
  const float sf = (float)s, off_lo = -1032.0f * sf, off_hi = -72.0f * sf;       // exact: 11 bits times 11 and 4
  half2_t h[4];                                             // codes (0,4) (1,5) (2,6) (3,7)
#pragma unroll
  for (int p = 0; p < 2; ++p) {
    const uint32_t src = p ? q >> 8 : q;
    h[2 * p] = __builtin_bit_cast(half2_t, (src & 0x000F000Fu) | 0x64006400u);
    h[2 * p + 1] = __builtin_bit_cast(half2_t, (src & 0x00F000F0u) | 0x54005400u);
  }
  auto weight = [&](int e) { return fmaf((float)h[e & 3][e >> 2], sf, e & 1 ? off_hi : off_lo); };
  u32x4 o;
#pragma unroll
  for (int w = 0; w < 4; ++w) {
    const float2_t f = {weight(2 * w), weight(2 * w + 1)};
    o[w] = __builtin_bit_cast(uint32_t, __builtin_convertvector(f, bf16x2_t));
  }
  return __builtin_bit_cast(bf16x8_t, o);
}

// MODE as in small_m_kernel; BF16 (bf16 tile type) exists for SM_PLAIN only, which serves every group size.
// DUAL: the -eps forward reads activations of its own (x2): one pass over the codes, two dense products.
// TILE_ROUND: the sensitive weights enter as v +- eps z rounded to the tile type, as they stand in the tiled
// kernel's weight tile (the dense code under them is the zero code), instead of v and z rounded one by one: for the
// layers whose other kernel is the tiled one, so that both give the same results up to fp32 summation order.
// Accumulator sets:            one set of x                       two sets (DUAL)
//   v and z apart              0: dense + x v^T  1: x z^T         0, 1: the same of x   2, 3: of x2
//   TILE_ROUND                 0: dense  1: x w+^T  2: x w-^T     0: dense + x w+^T     1: dense + x w-^T of x2
//   TILE_ROUND, ONE sign       0: dense + x w+^T
template <bool DUAL, bool TILE_ROUND, bool ONE> constexpr int split_sets() { return TILE_ROUND ? (ONE ? 1 : DUAL ? 2 : 3) : (DUAL ? 4 : 2); }
template <int MODE, bool DUAL, bool TILE_ROUND> constexpr int split_max_waves() {
  return MODE == SM_LUT || DUAL || TILE_ROUND ? 8 : SP_MAX_WAVES;
}
// Floats of LDS per wave: its window of entries, then its x, then its accumulators of `subs` subtiles.
constexpr int split_wave_floats(int nacc, int subs) {
  const int acc = nacc * subs * 256, x = (16 * SP_XROW * 2 + 15) / 16 * 4;
  return acc > x ? acc : x;
}
// SUBS: the workgroup's 16-row subtiles of the band.   XP: load instructions for 16 token rows of x, four rows each; with
// XP = 1 rows 4..15 of the operands are whatever LDS held: they only reach output rows that do not exist.
template <int MODE, bool BF16, bool DUAL, bool TILE_ROUND, bool ONE, bool BEHIND, int SUBS, int XP>
__device__ __forceinline__ void band_split_body(const SmallArgs& a, const small_words tab, int index, const int bid, const int slice) {
  static_assert(!BF16 || (MODE == SM_PLAIN && TILE_ROUND), "bf16 tile: plain dequantisation, rounded as in the tile");
  constexpr bool FAST = MODE == SM_FAST, LUT = MODE == SM_LUT;
  static_assert(!ONE || (TILE_ROUND && !DUAL), "instantiations");
  constexpr int SETS = DUAL ? 2 : 1;
  constexpr int NACC = split_sets<DUAL, TILE_ROUND, ONE>();
  constexpr int RED = split_wave_floats(NACC, SUBS);
  // The entries stand behind the first block of the codes where one window holds them all: their bounds, values and columns of x are a
  // chain of memory round trips that the block's dequantisation covers.  Single forwards of TILE_ROUND layers, us: a 5000 x 4160 layer with
  // the bf16 tile at 77 tokens 20.8 -> 19.5, 4096 x 4096 at 128 20.1 -> 18.7.  Elsewhere before all codes: groups of 128 have less to
  // dequantise (six forwards of an OPT block at one token 53.1 -> 53.9), and with both signs rounded the registers of the block and of the
  // entries together cost a workgroup per CU (one Mistral block with the bf16 tile at 40 tokens 87 -> 99).
  constexpr bool LATER = TILE_ROUND && ONE;
  constexpr int DENSE1 = TILE_ROUND ? 1 : 2;                // accumulator set of x2's dense product
  typedef SplitOps<BF16> Ops;
  typedef typename Ops::frag frag_t;
  extern __shared__ __attribute__((aligned(16))) float red[];                     // [waves][RED]

  asm volatile("" : "+s"(index));                           // (the bodies read the entry one by one: read before the choice, it overflows the scalar registers)
  const SmallMat mt = read_matrix(tab, index);
  if (slice * SM_ROWS >= mt.M) return;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), waves = (int)blockDim.x >> 6;
  const int N = mt.N, K = mt.K, M = min(SM_ROWS, mt.M - slice * SM_ROWS);
  // this workgroup's rows: SUBS of the four 16-row subtiles of a band, from subtile sub0 on
  constexpr int PIECES = 4 / SUBS;
  const int band = (bid - mt.first_block) / PIECES, piece = (bid - mt.first_block) % PIECES, sub0 = piece * SUBS, ktiles = K >> 6;
  const size_t row0 = (size_t)slice * SM_ROWS;
  const auto g_x = SZO_GLOBAL(uint16_t, mt.x) + row0 * (size_t)K;
  const auto g_x2 = SZO_GLOBAL(uint16_t, DUAL ? mt.x2 : mt.x) + row0 * (size_t)K;
  const auto g_q = SZO_GLOBAL(uint8_t, mt.qweight) + (size_t)band * (size_t)ktiles * 2048 + 512 * sub0;
  const auto g_scales = SZO_GLOBAL(uint16_t, mt.scales);
  const auto g_tile_ptr = SZO_GLOBAL(uint32_t, mt.tile_ptr) + (size_t)band * (size_t)ktiles;
  const auto g_sp_idx = SZO_GLOBAL(uint32_t, mt.sp_idx);
  const auto g_sp_val = SZO_GLOBAL(float, mt.sp_val);
  const auto g_target = SZO_GLOBAL(uint16_t, mt.target) + row0 * (size_t)N;
  float __attribute__((address_space(1)))* const g_y = (float __attribute__((address_space(1)))*)mt.y + row0 * (size_t)N;
  const int nn = lane & 15, jj = lane >> 4;
  const bool with_z = a.eps != 0.0f;

  // this wave's part of K, in blocks of 128 columns (the last block of a K that is an odd multiple of 64 is half
  // empty: its codes are read from the last tile and multiplied with zeros)
  const int nkb = (K + 127) >> 7;
  const int b0 = wave * nkb / waves, b1 = (wave + 1) * nkb / waves;

  // x of a block, 16 rows of 256 bytes, is loaded row by row (16 lanes per row: one load instruction touches 8 lines,
  // against 64 if every lane fetched the pieces of its own operand row) and turned into operands through 4 KB of
  // LDS of the wave's own; rows past M repeat the last one and only reach output rows past M.
  const int xr_row = lane >> 4, xr_piece = lane & 15;       // load i: row 4 i + xr_row, columns 8 xr_piece ..
  const uint32_t row_bytes = (uint32_t)K * 2u, last_row = (uint32_t)(M - 1) * row_bytes;
  const uint32_t xrow = min((uint32_t)nn * row_bytes, last_row);   // operand row of this lane (sensitive entries), in bytes
  u32x4 q[SUBS], xr[SETS][XP] = {};
  // Loads are a uniform base plus a 32-bit byte offset per lane (64-bit addresses per lane cost twice the registers).
  const auto b_x = (const uint8_t __attribute__((address_space(1)))*)g_x;
  const auto b_x2 = (const uint8_t __attribute__((address_space(1)))*)g_x2;
  const uint32_t q_lane = (uint32_t)nn * 32u + (uint32_t)(jj & 1) * 16u;
  auto load_q = [&](int b, int s) {
    const uint32_t off = (uint32_t)min(2 * b + (jj >> 1), ktiles - 1) * 2048u + q_lane;
    q[s] = *reinterpret_cast<const u32x4 __attribute__((address_space(1)))*>(g_q + (size_t)off + 512 * s);
  };
  const uint32_t x_lane = (uint32_t)xr_row * row_bytes;
  auto load_x = [&](int b) {
    const uint32_t col = (uint32_t)min(128 * b + 8 * xr_piece, K - 8) * 2u;
#pragma unroll
    for (int i = 0; i < XP; ++i)
#pragma unroll
      for (int set = 0; set < SETS; ++set)
        xr[set][i] = *reinterpret_cast<const u32x4 __attribute__((address_space(1)))*>(
            (set ? b_x2 : b_x) + (size_t)(min(x_lane + (uint32_t)(4 * i) * row_bytes, last_row) + col));
  };
  const int gshift = mt.group_shift, groups = FAST ? K >> 7 : LUT ? 0 : K >> gshift;
  const auto g_sc = (const uint8_t __attribute__((address_space(1)))*)(g_scales + (size_t)band * (size_t)groups * 64);
  uint64_t sc = 0u;                                         // the lane's scales of a group, subtile sub0's first
  auto load_scales = [&](int b) {
    if (LUT) return;
    const int g = FAST ? b : min((128 * b + 32 * jj) >> gshift, groups - 1);
    sc = *reinterpret_cast<const uint64_t __attribute__((address_space(1)))*>(g_sc + (size_t)((uint32_t)g * 128u + 8u * (uint32_t)nn));
  };
  uint32_t e_lo = 0, e_hi = 0;                              // this wave's sensitive entries
  if (b0 < b1) {
    const small_words bounds = (small_words)(uintptr_t)g_tile_ptr;       // scalar loads: a vector load is waited for behind the codes (the six calls 55.4 -> 54.1)
    auto load_bounds = [&]() {
      if (mt.nnz > 0) { e_lo = bounds[2 * b0]; e_hi = bounds[min(2 * b1, ktiles)]; }
    };
    if (!BEHIND) load_bounds();
#pragma unroll
    for (int s = 0; s < SUBS; ++s) load_q(b0, s);
    load_x(b0);
    load_scales(b0);
    if (BEHIND) load_bounds();
  }
  uint32_t tb[LUT ? SUBS : 1][8];
  if (LUT) {
#pragma unroll
    for (int s = 0; s < (LUT ? SUBS : 1); ++s) load_lut_planes(g_scales + (size_t)min(band * 64 + 16 * (sub0 + s) + nn, N - 1) * 16, tb[s]);
  }

  float4_t acc[NACC][SUBS];
#pragma unroll
  for (int i = 0; i < NACC; ++i)
#pragma unroll
    for (int s = 0; s < SUBS; ++s) acc[i][s] = float4_t{0.0f, 0.0f, 0.0f, 0.0f};

  // ---- dense: this wave's blocks of 128 columns, codes and x one block ahead ----
  uint16_t* const xs = reinterpret_cast<uint16_t*>(red + wave * RED);              // [16][SP_XROW], in place of the window
  uint32_t magic_lo = 0x64006400u, magic_hi = 0x54005400u;
  asm volatile("" : "+v"(magic_lo), "+v"(magic_hi));
  const half8_t minus_offsets = {(_Float16)-1032.0f, (_Float16)-1032.0f, (_Float16)-72.0f, (_Float16)-72.0f,
                                 (_Float16)-1032.0f, (_Float16)-1032.0f, (_Float16)-72.0f, (_Float16)-72.0f};
  // MORE at compile time: as a run-time condition around the loads it made the compiler drain them in every iteration
  auto dense_block = [&](int b, auto more_tag) {
    constexpr bool MORE = decltype(more_tag)::value;
    const bool empty = 128 * b + 8 * xr_piece >= K;         // the columns this lane has loaded lie past the end of K
    frag_t af[SETS][4];
#pragma unroll
    for (int set = 0; set < SETS; ++set) {
#pragma unroll
      for (int i = 0; i < XP; ++i)
        *reinterpret_cast<frag_t*>(xs + (4 * i + xr_row) * SP_XROW + 8 * xr_piece) =
            Ops::activations(empty ? u32x4{0u, 0u, 0u, 0u} : xr[set][i]);
      asm volatile("" ::: "memory");                        // written by the wave's other lanes; LDS keeps a wave's order
#pragma unroll
      for (int t = 0; t < 4; ++t) af[set][t] = *reinterpret_cast<const frag_t*>(xs + nn * SP_XROW + 32 * jj + 8 * t);
      asm volatile("" ::: "memory");
    }
    if (MORE) load_x(b + 1);
    const half4_t sh4 = __builtin_bit_cast(half4_t, SUBS == 4 ? sc : sc >> (16 * sub0));
    if (MORE) load_scales(b + 1);
    float4_t init[SETS];
#pragma unroll
    for (int set = 0; set < SETS; ++set) {
      init[set] = float4_t{0.0f, 0.0f, 0.0f, 0.0f};
      if constexpr (FAST) {
#pragma unroll
        for (int t = 0; t < 4; ++t) init[set] = Ops::dense(af[set][t], minus_offsets, init[set]);
      }
    }
#pragma unroll
    for (int s = 0; s < SUBS; ++s) {
      const u32x4 qs = q[s];
      if (MORE) load_q(b + 1, s);
      float4_t tmp[SETS];
#pragma unroll
      for (int set = 0; set < SETS; ++set) tmp[set] = FAST ? init[set] : acc[set * DENSE1][s];
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        frag_t w;
        if constexpr (BF16) w = dequant_word_bf16(qs[t], sh4[s]);
        else if constexpr (LUT) w = sm_lut_word(qs[t], tb[s]);
        else w = sm_dequant_word<FAST>(qs[t], magic_lo, magic_hi, half2_t{sh4[s], sh4[s]});
#pragma unroll
        for (int set = 0; set < SETS; ++set) tmp[set] = Ops::dense(af[set][t], w, tmp[set]);
      }
#pragma unroll
      for (int set = 0; set < SETS; ++set) {
        if (FAST) {
          const float sf = (float)sh4[s];
#pragma unroll
          for (int r = 0; r < 4; ++r) acc[set * DENSE1][s][r] = fmaf(tmp[set][r], sf, acc[set * DENSE1][s][r]);
        } else {
          acc[set * DENSE1][s] = tmp[set];
        }
      }
      __builtin_amdgcn_sched_barrier(0);                    // subtiles in program order: fewer registers in flight
    }
  };
  // ---- sensitive entries: 128 at a time into LDS of the wave's own, then 16 per matrix product ----
  auto sensitive_entries = [&]() {
    uint32_t* const wk = reinterpret_cast<uint32_t*>(LATER ? red + waves * RED + wave * SP_WIN_FLOATS : red + wave * RED);      // column
    uint16_t* const wr = reinterpret_cast<uint16_t*>(wk + SP_WIN);                  // row of the band
    uint16_t* const wv = wr + SP_WIN;                                                // 16-bit v | v + eps z
    uint16_t* const wz = wv + SP_WIN;                                                // 16-bit z | v - eps z
    for (uint32_t w0 = e_lo & ~3u; w0 < e_hi; w0 += SP_WIN) {
      const uint32_t j = w0 + 2u * lane, last = mt.nnz - 1u;
      uint32_t idx[2];
      float val[2], z[2] = {0.0f, 0.0f};
#pragma unroll
      for (int e = 0; e < 2; ++e) {
        const uint32_t je = min(j + e, last);               // clamped; entries past the end are left out
        idx[e] = g_sp_idx[je];
        val[e] = g_sp_val[je];
      }
      if (with_z) zbar_pair((mt.nnz_base + j) >> 2, (j & 2u) != 0u, a.seed, a.step, z);
      // A part of a band keeps those of its own rows, one after the other, in order; a whole band keeps all of them where they
      // stand and counts those of this wave's columns, lo .. hi of the window.
      uint32_t row[2], at = SUBS == 4 ? 2u * lane : 0u;
      uint32_t lo = SUBS == 4 ? max(e_lo, w0) - w0 : 0u, hi = SUBS == 4 ? min(e_hi - w0, (uint32_t)SP_WIN) : 0u;
      bool in[2];
#pragma unroll
      for (int e = 0; e < 2; ++e) {
        const uint32_t n = sm_fast_div(idx[e], mt.div_mul, mt.div_shift);
        row[e] = n - (uint32_t)(band * 64 + 16 * sub0);
        idx[e] -= n * (uint32_t)K;
        in[e] = SUBS == 4 || (j + e >= e_lo && j + e < e_hi && row[e] < (uint32_t)(16 * SUBS));
        if (SUBS < 4) {
          const uint64_t m = __ballot(in[e]);
          at += __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
          hi += (uint32_t)__popcll(m);
        }
      }
#pragma unroll
      for (int e = 0; e < 2; ++e) {
        if (in[e]) {
          wk[at] = idx[e];
          wr[at] = (uint16_t)row[e];
          wv[at] = Ops::narrow(TILE_ROUND ? fmaf(a.eps, z[e], val[e]) : val[e]);
          wz[at] = Ops::narrow(TILE_ROUND ? fmaf(-a.eps, z[e], val[e]) : z[e]);
          ++at;
        }
      }
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");     // window visible to the other lanes of the wave
      for (uint32_t g0 = 0; g0 < hi; g0 += 16u) {
        const uint32_t at = g0 + 4u * (uint32_t)jj;
        const u32x4 kw = *reinterpret_cast<const u32x4*>(wk + at);
        const u32x2 rw = *reinterpret_cast<const u32x2*>(wr + at);
        const u32x2 vw = *reinterpret_cast<const u32x2*>(wv + at);
        const u32x2 zw = *reinterpret_cast<const u32x2*>(wz + at);
        uint32_t mlo[4], mhi[4];
        uint16_t ax[SETS][4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {                       // every gather requested before the first is used
          const uint32_t e = at + (uint32_t)i, col = e >= lo && e < hi ? kw[i] : 0u;   // not an entry of this wave: a valid address, masked below
#pragma unroll
          for (int set = 0; set < SETS; ++set)
            ax[set][i] = *reinterpret_cast<const uint16_t __attribute__((address_space(1)))*>(
                (set ? b_x2 : b_x) + (size_t)(xrow + 2u * col));
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          one_hot_entry((rw[i >> 1] >> (16 * (i & 1))) & 63u, nn, at + (uint32_t)i >= lo && at + (uint32_t)i < hi, mlo[i], mhi[i]);
#pragma unroll
          for (int set = 0; set < SETS; ++set) ax[set][i] = Ops::activation(ax[set][i]);
        }
        u32x2 xw[SETS];
#pragma unroll
        for (int set = 0; set < SETS; ++set)
          xw[set] = u32x2{(uint32_t)ax[set][0] | ((uint32_t)ax[set][1] << 16), (uint32_t)ax[set][2] | ((uint32_t)ax[set][3] << 16)};
#pragma unroll
        for (int s = 0; s < SUBS; ++s) {
          u32x2 bv, bz;
#pragma unroll
          for (int h = 0; h < 2; ++h) {
            const uint32_t ma = (s < 2) ? mlo[2 * h] : mhi[2 * h], mb = (s < 2) ? mlo[2 * h + 1] : mhi[2 * h + 1];
            const uint32_t mask = __builtin_amdgcn_perm(mb, ma, (s & 1) ? 0x07060302u : 0x05040100u);
            bv[h] = vw[h] & mask;
            bz[h] = zw[h] & mask;
          }
          if constexpr (TILE_ROUND) {
            constexpr int PLUS = DUAL || ONE ? 0 : 1;
            acc[PLUS][s] = Ops::sparse(xw[0], bv, acc[PLUS][s]);
            if constexpr (!ONE) acc[PLUS + 1][s] = Ops::sparse(xw[SETS - 1], bz, acc[PLUS + 1][s]);
          } else {
#pragma unroll
            for (int set = 0; set < SETS; ++set) {
              acc[2 * set][s] = Ops::sparse(xw[set], bv, acc[2 * set][s]);
              if (with_z) acc[2 * set + 1][s] = Ops::sparse(xw[set], bz, acc[2 * set + 1][s]);
            }
          }
        }
      }
      asm volatile("" ::: "memory");                        // the next refill overwrites the window
    }
  };

  int next = b0;
  if (LATER && e_hi - e_lo <= (uint32_t)SP_WIN && next + 1 < b1) dense_block(next++, std::true_type{});
  sensitive_entries();
  for (; next + 1 < b1; ++next) dense_block(next, std::true_type{});
  if (b0 < b1) dense_block(b1 - 1, std::false_type{});

  // ---- sum over the waves, in wave order ----
  {
    float4_t* const mine = reinterpret_cast<float4_t*>(red + wave * RED);
#pragma unroll
    for (int i = 0; i < NACC; ++i)
#pragma unroll
      for (int s = 0; s < SUBS; ++s) mine[i * 64 * SUBS + s * 64 + lane] = acc[i][s];
  }
  __syncthreads();
  // Output o: column o & 15 of subtile o >> 8, token row (o >> 4) & 15; its accumulator sits in register m & 3 of lane
  // 16 (m >> 2) + column.  Wave-wide LDS reads touch every bank once, y is stored 64 bytes at a time.
  double lp = 0.0, lm = 0.0;
  bool all_finite = true;
  // AGAIN: a second time, with the outputs of token rows that hold an infinite or NaN activation by their definition
  auto finish = [&](auto again_tag) {
    constexpr bool AGAIN = decltype(again_tag)::value;
    WeightSource source;
    global_u16 x_plus, x_minus;
    if constexpr (AGAIN) {
      int again = index;                                    // the entry is read again (laundered: not kept for this)
      asm volatile("" : "+s"(again));
      const SmallMat ms = read_matrix(tab, again);
      source = WeightSource{(global_u8)ms.qweight, LUT ? nullptr : (global_u16)ms.scales, LUT ? (global_u16)ms.scales : nullptr,
                            (global_u32)ms.tile_ptr, (global_u32)ms.sp_idx, (global_f32)ms.sp_val, ms.K, ms.group_shift,
                            ms.nnz, ms.nnz_base, a.seed, a.step};
      x_plus = (global_u16)ms.x + (size_t)slice * SM_ROWS * (size_t)ms.K;
      x_minus = (global_u16)(DUAL ? ms.x2 : ms.x) + (size_t)slice * SM_ROWS * (size_t)ms.K;
    }
    lp = 0.0; lm = 0.0;
    for (int o = tid; o < 256 * SUBS; o += (int)blockDim.x) {
      const int m = (o >> 4) & 15, n = band * 64 + 16 * (sub0 + (o >> 8)) + (o & 15);
      if (m >= M || n >= N) continue;
      const float* p = red + (o >> 8) * 256 + ((m >> 2) * 16 + (o & 15)) * 4 + (m & 3);
      float t = 0.0f;
      if (a.loss_mode) t = __uint_as_float((uint32_t)g_target[(size_t)m * N + n] << 16);
      float d[NACC];
#pragma unroll
      for (int i = 0; i < NACC; ++i) d[i] = 0.0f;
      for (int w = 0; w < waves; ++w, p += RED) {
#pragma unroll
        for (int i = 0; i < NACC; ++i) d[i] += p[i * SUBS * 256];
      }
      float yp, ym;
      if (TILE_ROUND) {
        yp = DUAL || ONE ? d[0] : d[0] + d[1 % NACC];
        ym = DUAL ? d[NACC - 1] : ONE ? yp : d[0] + d[NACC - 1];
      } else {
        yp = d[0] + a.eps * d[NACC > 1 ? 1 : 0];
        ym = d[NACC > 1 ? NACC - 2 : 0] - a.eps * d[NACC - 1];
      }
      if constexpr (AGAIN) {
        constexpr int DT = BF16 ? SZO_TILE_BF16 : SZO_TILE_F16;
        nonfinite_output<DT>(source, x_plus + (size_t)m * source.K, (uint32_t)n, a.eps, yp);
        nonfinite_output<DT>(source, x_minus + (size_t)m * source.K, (uint32_t)n, -a.eps, ym);
      } else {
        all_finite = all_finite && __builtin_isfinite(yp) && __builtin_isfinite(ym);
      }
      if (a.loss_mode) {
        const float dp = yp - t, dm = ym - t;
        lp += (double)(dp * dp);
        lm += (double)(dm * dm);
      }
      if (!DUAL && a.store_sign) g_y[(size_t)m * N + n] = a.store_sign > 0 ? yp : ym;
    }
  };
  finish(std::false_type{});
  if (__builtin_expect(!__all(all_finite), 0)) finish(std::true_type{});
  if (a.loss_mode) {
    __shared__ double part[2][SP_MAX_WAVES];
    lp = wave_sum(lp);
    lm = wave_sum(lm);
    if (lane == 0) { part[0][wave] = lp; part[1][wave] = lm; }
    __syncthreads();
    if (tid == 0) {
      double bp = 0.0, bm = 0.0;
      for (int w = 0; w < waves; ++w) { bp += part[0][w]; bm += part[1][w]; }
      const int pi = mt.partial_base + (slice * ((N + 63) >> 6) + band) * PIECES + piece;
      ((double __attribute__((address_space(1)))*)a.partial_plus)[pi] = bp * mt.loss_scale;
      ((double __attribute__((address_space(1)))*)a.partial_minus)[pi] = bm * mt.loss_scale;
    }
  }
}

// ONE: the "+" forward alone is wanted (single forwards of TILE_ROUND layers); the partials and outputs of the other are not valid then.
// What a wave needs before it can ask for its matrix's table entry comes as arguments of its own, ahead of the rest: they
// are in scalar registers when the wave starts (kernarg preload, see build.py), so that the entry is the first memory round trip and
// not the third, behind the arguments and the size of the grid.  us per pass over four sets of weights: a step over one small layer 11.30 -> 10.97,
// six calls over an OPT block at one token 57.6 -> 55.4, a step over it at 16 tokens 44.0 -> 43.4.
// BEHIND: a wave asks for its tile bounds behind its first block's loads (see launch_mode).
struct SplitArgs { const SmallMat* table; int n_mats; uint32_t part_shifts; int slices, few_rows, workgroups; SmallArgs a; };   // as the arguments lie in memory
template <int MODE, bool BF16, bool DUAL, bool TILE_ROUND, bool ONE, bool BEHIND>
__global__ void __launch_bounds__((64 * split_max_waves<MODE, DUAL, TILE_ROUND>()))
band_split_kernel(const SmallMat* table, int n_mats, uint32_t part_shifts, int slices, int few_rows, int workgroups, SmallArgs a) {
  int bid = xcd_unit((int)blockIdx.x, workgroups);
  const small_words tab = table ? (small_words)table
                                : (small_words)__builtin_amdgcn_kernarg_segment_ptr() + (offsetof(SplitArgs, a) + offsetof(SmallArgs, inl)) / 4;
  const int slice = bid % slices;
  bid /= slices;
  const int index = find_index(tab, n_mats, bid);
  const uint32_t part_shift = (part_shifts >> (4 * (index & 7))) & 15u;
  auto run = [&](auto rows_tag) {
    constexpr int XP = decltype(rows_tag)::value;
    if (part_shift == 0) band_split_body<MODE, BF16, DUAL, TILE_ROUND, ONE, BEHIND, 4, XP>(a, tab, index, bid, slice);
    else if (part_shift == 1) band_split_body<MODE, BF16, DUAL, TILE_ROUND, ONE, BEHIND, 2, XP>(a, tab, index, bid, slice);
    else band_split_body<MODE, BF16, DUAL, TILE_ROUND, ONE, BEHIND, 1, XP>(a, tab, index, bid, slice);
  };
  if (MODE == SM_FAST && !DUAL && few_rows) run(std::integral_constant<int, 1>{});
  else run(std::integral_constant<int, 4>{});
}

template <int MODE, bool BF16, bool DUAL, bool TILE_ROUND, bool ONE = false, bool BEHIND = false>
static int launch(const SplitLaunch& l, const SmallArgs& a, hipStream_t stream) {
  constexpr int nacc = split_sets<DUAL, TILE_ROUND, ONE>(), most = split_max_waves<MODE, DUAL, TILE_ROUND>();
  constexpr size_t window = (TILE_ROUND && ONE ? SP_WIN_FLOATS : 0) * sizeof(float), most_bytes = (split_wave_floats(nacc, 4) * sizeof(float) + window) * most;
  const int waves = l.waves < most ? l.waves : most;
  static std::atomic<uint64_t> lds_limit_set{0};             // per instantiation
  const auto kern = band_split_kernel<MODE, BF16, DUAL, TILE_ROUND, ONE, BEHIND>;
  const int rc = set_lds_limit_once(lds_limit_set, (const void*)kern, most_bytes);
  if (rc != SZO_OK) return rc;
  kern<<<(unsigned)l.workgroups, 64 * waves, (split_wave_floats(nacc, l.subs) * sizeof(float) + window) * (size_t)waves, stream>>>(a.table, a.n_mats, a.part_shifts, a.slices, a.few_rows, l.workgroups, a);
  SZO_LAUNCH_CHECK();
  return SZO_OK;
}

// The bf16 form for two sets of activations: with the bounds in front of the loads the compiler gives it 21 registers less and orders its
// products one behind the other, which large launches lose by; small ones and short K lose by the later bounds.  us per step, in front / behind:
// four Llama blocks at 3 / 16 / 40 tokens 138 / 215 / 424, 133 / 208 / 416, one at 16 (664 workgroups) 64.0 / 62.8, 8192 x 4096 at 64 (512) 40.7 / 39.5,
// 4096 x 8192 at 120 (512) 67.1 / 65.4; on the other side 8192 x 1024 at 110 (896) 33.3 / 34.2, 4096 x 1024 / 4096 at 64 (256) 13.2 / 13.4, 22.8 / 22.7,
// 8192 x 8192 at 2 (256) 19.6 / 20.0.  The other forms are the same either way, or gain 1 to 3 % in front.
static bool bounds_behind(const SplitLaunch& l) { return l.workgroups >= 512 && l.longest_k >= 2048; }
template <bool DUAL>
static int launch_mode(const SplitLaunch& l, const SmallArgs& a, hipStream_t stream) {
  if constexpr (!DUAL) {
    if (l.bf16 && l.one) return launch<SM_PLAIN, true, false, true, true>(l, a, stream);
    if (l.tile_round && l.one) return launch<SM_PLAIN, false, false, true, true>(l, a, stream);
  }
  if constexpr (DUAL) {
    if (l.bf16 && bounds_behind(l)) return launch<SM_PLAIN, true, true, true, false, true>(l, a, stream);
  }
  if (l.bf16) return launch<SM_PLAIN, true, DUAL, true>(l, a, stream);
  if (l.tile_round) return launch<SM_PLAIN, false, DUAL, true>(l, a, stream);
  if (l.mode == SM_FAST) return launch<SM_FAST, false, DUAL, false>(l, a, stream);
  if (l.mode == SM_LUT) return launch<SM_LUT, false, DUAL, false>(l, a, stream);
  return launch<SM_PLAIN, false, DUAL, false>(l, a, stream);
}

int split_launch(const SplitLaunch& l, const SmallArgs& a, hipStream_t stream) {
  return l.dual ? launch_mode<true>(l, a, stream) : launch_mode<false>(l, a, stream);
}

}  // namespace szo
