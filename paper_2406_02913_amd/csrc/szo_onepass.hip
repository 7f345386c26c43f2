// A whole step's forwards with ONE dense product per layer, on the matrix cores.
//
// Both forwards of a layer of szo_zo_step read the same activations, and the sensitive weights of the two are
// v + eps z and v - eps z (Section 3.4), so
//     D = x (Dequantize(Q(w_dense)) + v)^T        Z = x z^T        y(+-) = D +- eps Z:
// the dense product is the same in both and is computed once; the sensitive entries add products with a matrix that has
// a few entries per 64 rows and 128 columns.
//
// Workgroup = 64 token rows x 256 rows of W, four waves, each one band of 64 rows of W by itself: a wave streams its
// codes into registers and dequantises them there into operands of v_mfma_f32_32x32x16 (every operand serves two
// blocks of 32 token rows), so the weights never pass through LDS and only the activations, converted once per
// workgroup and shared by its waves, need a barrier (one per chunk of 128 columns, double buffered).  Two workgroups
// share a CU and cover each other's barriers.
//
// Sensitive entries.  A wave keeps a ring of its band's entries in LDS, 256 computed at a time.  Sixteen of them at a
// time are written as two one-hot 64 x 16 operands (v and z at [row][slot]) to LDS of the wave's own; the wave gathers
// their columns of the staged x and multiplies both: D += x_g V^T, Z += x_g Z^T.  The first sixteen of a chunk (at a
// density of 0.1 % it has eight on average) run inside the dense schedule, more of them in a loop behind it.
//
// Precision.  fp16 tile, groups of 128 (GROUP_SCALE, one group per chunk): the integer codes are multiplied exactly and
// the sum of a chunk takes the group's scale in fp32, as in the few-token kernels; other groups, and the bf16 tile: the
// dense weights are rounded to the tile type as in the tiled kernel.  v and z are rounded to it one by one (2^-11 relative
// in fp16) instead of as part of w +- eps z, and eps is applied in fp32.
// Relative error of a loss against fp64, two Llama blocks at 128 tokens: 4e-9 with GROUP_SCALE (few-token kernel 8e-9,
// weights rounded after scaling 7e-8); of g, 6e-4 in all three.
// GROUP_SCALE needs a third set of sums: it takes one block of 32 rows of W after the other (the operands of x are
// read twice, the scales cost 64 instructions per chunk instead of 64 in the dequantisation) and holds half as much of x
// in registers.  us per step, weights rounded after scaling -> scale in fp32: one Llama block with SZO_STEP_ONE_DENSE_PASS at 4096 tokens
// 2182 -> 2126, four Llama blocks at 128 tokens 322 -> 316, eight OPT blocks at 64 325 -> 327, a 1024 x 4096 layer with
// outputs at 300 tokens (20 workgroups: nothing stands behind the scaling of a chunk) 65.2 -> 66.9.
#include <algorithm>
#include <cstddef>
#include <type_traits>
#include <vector>
#include "szo_internal.h"
#include "szo_nonfinite.h"
#include "szo_rng.h"
#include "szo_tile.h"

namespace szo {

typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));

constexpr int OP_BM = 64, OP_BN = 256, OP_WAVES = 4;        // token rows, rows of W, waves of a workgroup
constexpr int OP_KC = 128;                                  // columns per chunk
constexpr int OP_XROW = 2 * OP_KC + 16;                     // LDS row of staged activations in bytes (+16 against bank conflicts)
constexpr int OP_RING = 512, OP_REFILL = 256;               // sensitive entries held / computed at a time per wave
constexpr int OP_TROW = 2 * OP_BN + 32;                     // LDS row of the target tile in the epilogue

struct OnePassLds {                                         // byte offsets
  static constexpr int X = 0, RING = X + 2 * OP_BM * OP_XROW, HOT = RING + OP_WAVES * OP_RING * 8,   // [wave] 2 x 64 rows x 16 slots
                       POS = HOT + OP_WAVES * 4096, SINK = POS + OP_WAVES * 64, BYTES = SINK + OP_WAVES * 256;
};
static_assert(OnePassLds::BYTES <= 80 * 1024 && OP_BM * OP_TROW <= OnePassLds::RING, "two workgroups per CU; the target tile replaces x");

__device__ __forceinline__ FwdParams read_entry(table_words e) {
  struct Words { uint32_t w[sizeof(FwdParams) / 4]; } raw;
#pragma unroll
  for (int i = 0; i < (int)(sizeof(FwdParams) / 4); ++i) raw.w[i] = e[i];
  return __builtin_bit_cast(FwdParams, raw);
}

// `entry`: where p came from in a descriptor table, or null if it came with the launch.
// SPARSE: most chunks of a band hold eight sensitive entries at most, whose gathers take half the slots of a group (see below).
template <int DT, bool STORE_Y, bool GROUP_SCALE, bool SPARSE>
__device__ __forceinline__ void onepass_body(const FwdParams& p, const int bid, table_words entry) {
  static_assert(!GROUP_SCALE || DT == SZO_TILE_F16, "integer codes are fp16 operands");
  typedef typename Frag<DT>::type frag_t;
  // Fields that are rarely needed are read again where they are used (the laundered pointer keeps the loads there).
  auto cold = [&]() -> FwdParams {
    if (entry == nullptr) return p;
    table_words e = entry;
    asm volatile("" : "+s"(e));
    return read_entry(e);
  };
  int bm, bn;
  tile_of_logical(logical_block(bid, p.grid_m * p.grid_n), p.grid_m, p.grid_n, 8, bm, bn);

  extern __shared__ __attribute__((aligned(16))) uint8_t smem[];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int m0 = bm * OP_BM, n0 = bn * OP_BN, K = p.K;
  const int ktiles = p.ktiles, nchunks = (K + OP_KC - 1) / OP_KC;
  const int band = n0 / 64 + wave;
  const int half = lane >> 5, l31 = lane & 31;

  // Scalar base plus 32 bits per lane, both pinned where they are used: left alone the compiler precomputes 64-bit lane
  // addresses for every load of the loop, which does not fit the register file.
  auto lane_address = [](global_u8 base, uint32_t lane_bytes) -> global_u8 {
    asm volatile("" : "+s"(base));
    asm volatile("" : "+v"(lane_bytes));
    return base + (size_t)lane_bytes;
  };

  // ---- codes and scales.  Lane (n, half) reads 16 bytes = 32 columns of row n (block j: row 32 j + n) of a 64-column
  //      tile; word w of them is the operand of columns 32 half + 8 w .. of the tile.  Tiles past the end re-read the last
  //      one and meet zeros in x; bands past N re-read the last band, their outputs are never used. ----
  const size_t bsafe = (size_t)min(band, p.bands - 1);
  const int gshift = p.group_shift;
  const global_u8 q_base = p.qweight + bsafe * (size_t)ktiles * 2048;
  const global_u8 s_base = (global_u8)(p.scales + bsafe * (size_t)(K >> gshift) * 64);
  const uint32_t q_lane = (uint32_t)l31 * 32u + (uint32_t)half * 16u;
  const uint32_t s_lane = (uint32_t)((l31 & 15) * 8 + (l31 >> 4) * 2);
  u32x4 q[2][2];                                            // [tile of the chunk][block of 32 rows of W]
  uint32_t sc[2][2];                                        // 32 bits each: packed in pairs, a load would be waited for where it is issued
  auto load_q = [&](int c, int t, int j) {
    const int k = min(2 * c + t, ktiles - 1);
    q[t][j] = *reinterpret_cast<global_u32x4>(lane_address(q_base + (size_t)k * 2048 + 1024 * j, q_lane));
    // group of columns 64 k + 32 half ..: with groups of 32 the two half waves read neighbouring groups
    const uint32_t h_off = gshift == 5 ? (uint32_t)half * 128u : 0u;
    if (!GROUP_SCALE) sc[t][j] = *reinterpret_cast<global_u16>(lane_address(s_base + (size_t)((k * 64) >> gshift) * 128 + 4 * j, s_lane + h_off));
  };
  auto load_group_scale = [&](int c, int j) {               // one per chunk: groups of 128
    sc[0][j] = *reinterpret_cast<global_u16>(lane_address(s_base + (size_t)min(c, (ktiles >> 1) - 1) * 128 + 4 * j, s_lane));
  };

  // ---- activations: thread tid stages 16 bytes of rows (tid / 16) + 16 i ----
  const global_u8 x_base = (global_u8)(p.x + (size_t)m0 * K);
  const uint32_t x_row = (uint32_t)(tid >> 4) * (uint32_t)K * 2u;      // in bytes; 64 rows of K < 2^23 columns (checked on the host)
  const uint32_t x_last = (uint32_t)min(p.M - 1 - m0, OP_BM - 1) * (uint32_t)K * 2u;
  constexpr int XP = GROUP_SCALE ? 2 : 4;                   // pieces of x in registers: half a chunk ahead, or a whole one
  u32x4 xr[XP];
  const int x_col = 8 * (tid & 15);
  auto load_x = [&](int c, int i) {
    const uint32_t col = (uint32_t)min(OP_KC * c + x_col, K - 8) * 2u;
    uint32_t row = x_row;                                   // (pinned: one register instead of one per piece)
    if (GROUP_SCALE) asm volatile("" : "+v"(row));
    xr[i % XP] = *reinterpret_cast<global_u32x4>(lane_address(x_base, min(row + (uint32_t)i * (uint32_t)K * 32u, x_last) + col));
  };
  u32x2 xo;
  auto clip_x = [&](int c) {                                // K an odd multiple of 64: the last chunk's second half is zero
    if (OP_KC * (c + 1) <= K) return;
#pragma unroll
    for (int i = 0; i < XP; ++i)
      if (OP_KC * c + x_col >= K) xr[i] = u32x4{0u, 0u, 0u, 0u};
  };
  auto store_x_word = [&](int c, int i, int w) {            // word w of piece i; every second one writes half the piece
    xo[w & 1] = stage_x_word<DT>(xr[i % XP], w);
    if (w & 1)
      *reinterpret_cast<u32x2*>(smem + OnePassLds::X + (c & 1) * OP_BM * OP_XROW + ((tid >> 4) + 16 * i) * OP_XROW + 16 * (tid & 15) + 8 * (w >> 1)) = xo;
  };

  float16_t acc[2][2], accz[2][2];                          // [block of 32 token rows][block of 32 rows of W]
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) { acc[i][j][r] = 0.0f; accz[i][j][r] = 0.0f; }

  // ---- sensitive entries ----
  const bool band_ok = band < p.bands && p.nnz > 0;
  u32x2* const ring = reinterpret_cast<u32x2*>(smem + OnePassLds::RING) + wave * OP_RING;    // v | z << 16 ; row << 8 | byte of the column
  uint8_t* const hot = smem + OnePassLds::HOT + wave * 4096;                                  // [v, z][64 rows][16 slots]; SPARSE: [v, z][half][64 rows][8 slots]
  uint32_t* const pos = reinterpret_cast<uint32_t*>(smem + OnePassLds::POS) + wave * 16;      // byte of the column of each slot
  uint8_t* const sink = smem + OnePassLds::SINK + wave * 256 + 4 * lane;
  const table_words bounds = (table_words)(uintptr_t)(p.tile_ptr + (band_ok ? (size_t)band * (size_t)ktiles : 0));       // scalar loads
  auto tp_at = [&](int c) -> uint32_t { return band_ok ? bounds[min(2 * c, ktiles)] : 0u; };
  uint32_t j_lo = tp_at(0), j_hi = tp_at(1);                // entries of the chunk
  uint32_t w_hi = 0;                                        // entries below w_hi have been computed
  auto refill = [&]() {                                     // only reached when an entry of the band is wanted: nnz > 0
    const FwdParams pr = cold();
    const uint32_t j = w_hi + 4u * lane, lastj = pr.nnz - 1u;
    uint32_t idx[4];
    float val[4], z[4] = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const uint32_t je = min(j + e, lastj);                // clamped; entries past the end are never consumed
      idx[e] = pr.sp_idx[je];
      val[e] = pr.sp_val[je];
    }
    if (pr.signed_eps != 0.0f) zbar_quad((pr.nnz_base + j) >> 2, pr.seed, pr.step, z);
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const uint32_t n = fast_div(idx[e], pr.div_mul, pr.div_shift);
      const uint32_t k = idx[e] - n * (uint32_t)pr.K, r = (n - (uint32_t)(band * 64)) & 63u;
      const uint32_t kb = 2u * ((k & (uint32_t)(OP_KC - 8)) + (uint32_t)lds_pos<DT>(0, (int)(k & 7u)));
      uint16_t vb, zb;
      Frag<DT>::store(&vb, val[e]);
      Frag<DT>::store(&zb, z[e]);
      ring[(j + e) & (uint32_t)(OP_RING - 1)] = u32x2{(uint32_t)vb | ((uint32_t)zb << 16), (r << 8) | kb};
    }
    w_hi += OP_REFILL;
  };
  // Group of up to 16 entries from entry g0.  Entry e of it stands in slot e, or, SPARSE, in slot e / 2 of half e & 1, so that
  // eight or fewer fill the first four slots of both halves and the columns of the others need not be gathered (two-byte
  // gathers of 32 rows meet on a quarter of the LDS banks).  Only the schedule's group looks whether it has eight: further
  // groups of a chunk are full but for the last, and a branch among their gathers keeps those of the second block of token rows from
  // running beside the products of the first.  Skipping a quarter at a time, or all of an empty group, spills registers in the
  // schedule (2.5 and 1.6 times as long).  What it gives, and where: kSparseEntries below.
  u32x2 ent = {0u, 0u};
  uint8_t* hot_at = sink;                                   // where this lane's last entry stands
  auto group_read = [&](uint32_t g0) { ent = ring[(g0 + (uint32_t)(lane & 15)) & (uint32_t)(OP_RING - 1)]; };
  auto group_put = [&](uint32_t g0, uint32_t g_end) {
    const bool mine = lane < 16 && g0 + (uint32_t)lane < g_end;
    *reinterpret_cast<uint16_t*>(hot_at) = 0;
    *reinterpret_cast<uint16_t*>(hot_at + (hot_at == sink ? 0 : 2048)) = 0;
    if constexpr (SPARSE) hot_at = mine ? hot + (ent[1] >> 8) * 16u + ((uint32_t)lane & 1u) * 1024u + ((uint32_t)lane >> 1) * 2u : sink;
    else hot_at = mine ? hot + (ent[1] >> 8) * 32u + 2u * (uint32_t)lane : sink;
    *reinterpret_cast<uint16_t*>(hot_at) = (uint16_t)(ent[0] & 0xFFFFu);
    *reinterpret_cast<uint16_t*>(mine ? hot_at + 2048 : sink) = (uint16_t)(ent[0] >> 16);
    // slots without an entry: a valid column, multiplied with zero
    *reinterpret_cast<uint32_t*>(lane < 16 ? (uint8_t*)(SPARSE ? pos + 8 * (lane & 1) + (lane >> 1) : pos + lane) : sink) = mine ? (ent[1] & 0xFFu) : 0u;
  };
  u32x4 gp[2], za[GROUP_SCALE ? 1 : 2], zb[2];              // (GROUP_SCALE: one block of token rows after the other)
  const uint32_t gather_base = (uint32_t)l31 * OP_XROW;
  auto group_pos = [&]() {
    gp[0] = *reinterpret_cast<const u32x4*>(pos + 8 * half);
    gp[1] = *reinterpret_cast<const u32x4*>(pos + 8 * half + 4);
  };
  uint16_t graw[8];
  bool many = false;                                        // SPARSE: more than eight entries in the schedule's group
  auto gather_all = [&](int c, int i) {
    const uint8_t* const x = smem + OnePassLds::X + (c & 1) * OP_BM * OP_XROW + 32 * i * OP_XROW;
#pragma unroll
    for (int e = 0; e < 8; ++e) graw[e] = *reinterpret_cast<const uint16_t*>(x + (gp[e >> 2][e & 3] + gather_base));
  };
  auto group_gather = [&](int c, int i) {                   // of the schedule
    if constexpr (SPARSE) {
      const uint8_t* const x = smem + OnePassLds::X + (c & 1) * OP_BM * OP_XROW + 32 * i * OP_XROW;
#pragma unroll
      for (int e = 0; e < 4; ++e) graw[e] = *reinterpret_cast<const uint16_t*>(x + (gp[0][e] + gather_base));
      if (many) {
#pragma unroll
        for (int e = 4; e < 8; ++e) graw[e] = *reinterpret_cast<const uint16_t*>(x + (gp[1][e - 4] + gather_base));
      } else {
#pragma unroll
        for (int e = 4; e < 8; ++e) graw[e] = 0;
      }
    } else {
      gather_all(c, i);
    }
  };
  auto group_pack = [&](int i) {
#pragma unroll
    for (int h = 0; h < 4; ++h) za[GROUP_SCALE ? 0 : i][h] = (uint32_t)graw[2 * h] | ((uint32_t)graw[2 * h + 1] << 16);
  };
  auto group_hot = [&](int which) {
#pragma unroll
    for (int j = 0; j < 2; ++j)
      zb[j] = *reinterpret_cast<const u32x4*>(SPARSE ? hot + which * 2048 + 1024 * half + (32 * j + l31) * 16 : hot + which * 2048 + (32 * j + l31) * 32 + 16 * half);
  };
  auto group_multiply = [&](int which, int i, int j) {
    float16_t& a = which ? accz[i][j] : acc[i][j];
    a = Frag<DT>::mfma(__builtin_bit_cast(frag_t, za[GROUP_SCALE ? 0 : i]), __builtin_bit_cast(frag_t, zb[j]), a);
  };
  auto group_all = [&](int c, uint32_t g0, uint32_t g_end) {
    while (w_hi < min(g0 + 16u, g_end)) refill();
    group_read(g0);
    group_put(g0, g_end);
    group_pos();
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      gather_all(c, i);
      group_pack(i);
#pragma unroll
      for (int which = 0; which < 2; ++which) {
        group_hot(which);
#pragma unroll
        for (int j = 0; j < 2; ++j) group_multiply(which, i, j);
      }
    }
  };

  // ---- dense operands ----
  DequantConsts dqk;
  dqk.magic_lo = 0x64006400u; dqk.magic_hi = 0x54005400u;
  asm volatile("" : "+v"(dqk.magic_lo), "+v"(dqk.magic_hi));
  u32x4 b[2][2];                                            // [parity of the step][block]; GROUP_SCALE: one block at a time, in [.][0]
  auto dequant = [&](int step, int j, int part) {           // words 2 part, 2 part + 1 of the operand of step 0..7
    const int t = (step >> 2) & 1, c = step & 3;
    const _Float16 sh = __builtin_bit_cast(_Float16, (uint16_t)sc[t][j]);
    if constexpr (DT == SZO_TILE_F16) {
      // as dequant_out, in plain C: the two words go side by side through the three instructions, so that none waits
      // for the one before it
      const uint32_t src = part ? q[t][j][c] >> 8 : q[t][j][c];
      half2_t lo = __builtin_bit_cast(half2_t, (src & 0x000F000Fu) | dqk.magic_lo);
      half2_t hi = __builtin_bit_cast(half2_t, (src & 0x00F000F0u) | dqk.magic_hi);
      lo = lo - half2_t{(_Float16)1032.0f, (_Float16)1032.0f};
      hi = hi - half2_t{(_Float16)72.0f, (_Float16)72.0f};
      if (!GROUP_SCALE) {
        lo = lo * half2_t{sh, sh};
        hi = hi * half2_t{sh, sh};
      }
      b[step & 1][GROUP_SCALE ? 0 : j][2 * part] = __builtin_bit_cast(uint32_t, lo);
      b[step & 1][GROUP_SCALE ? 0 : j][2 * part + 1] = __builtin_bit_cast(uint32_t, hi);
    } else {
#pragma unroll
      for (int w = 2 * part; w < 2 * part + 2; ++w)
        b[step & 1][j][w] = dequant_out<DT>(q[t][j][c], w, (float)sh, half2_t{sh, sh}, dqk);
    }
  };
  frag_t a[2][2];
  const uint32_t a_lane = (uint32_t)(OnePassLds::X + l31 * OP_XROW + 64 * half);
  auto read_a = [&](int c, int step, int i) {
    a[step & 1][i] = *reinterpret_cast<const frag_t*>(smem + a_lane + (c & 1) * OP_BM * OP_XROW + 32 * i * OP_XROW + 128 * ((step >> 2) & 1) + 16 * (step & 3));
  };

  // ---- prologue ----
#pragma unroll
  for (int i = 0; i < XP; ++i) load_x(0, i);
#pragma unroll
  for (int t = 0; t < 2; ++t)
#pragma unroll
    for (int j = 0; j < 2; ++j) load_q(0, t, j);
  *reinterpret_cast<u32x4*>(hot + 16 * lane) = u32x4{0u, 0u, 0u, 0u};
  *reinterpret_cast<u32x4*>(hot + 1024 + 16 * lane) = u32x4{0u, 0u, 0u, 0u};
  *reinterpret_cast<u32x4*>(hot + 2048 + 16 * lane) = u32x4{0u, 0u, 0u, 0u};
  *reinterpret_cast<u32x4*>(hot + 3072 + 16 * lane) = u32x4{0u, 0u, 0u, 0u};
  w_hi = j_lo & ~3u;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    if (!GROUP_SCALE && i == 0) clip_x(0);
#pragma unroll
    for (int w = 0; w < 4; ++w) store_x_word(0, i, w);
    load_x(i + XP < 4 ? 0 : min(1, nchunks - 1), (i + XP) & 3);
  }
#pragma unroll
  for (int j = 0; j < 2; ++j) {
    if (GROUP_SCALE) load_group_scale(0, j);
#pragma unroll
    for (int part = 0; part < 2; ++part) if (!GROUP_SCALE || j == 0) dequant(0, j, part);
  }
  __syncthreads();

  // ---- chunks of 128 columns: 8 steps of 16 columns x 4 matrix instructions.  Behind every instruction stands a share of
  //      the work for later: the next step's operands, the next chunk's activations, the entries' operands ----
  for (int c = 0; c < nchunks; ++c) {
    const uint32_t j_next = tp_at(c + 2);
    while (w_hi < min(j_lo + 16u, j_hi)) refill();
#pragma unroll
    for (int i = 0; i < 2; ++i) read_a(c, 0, i);
    group_read(j_lo);
    if (SPARSE) many = j_hi - j_lo > 8u;
    auto behind = [&](int s) {                              // what stands behind matrix instruction s of 32
      if (s == 4) group_put(j_lo, j_hi);
      if (s == 8) group_pos();
      if (GROUP_SCALE) {
        if (s == 11) group_gather(c, 0);
        if (s == 13) group_hot(0);
        if (s == 14) group_pack(0);
        if (s == 15 || s == 16) group_multiply(0, 0, s - 15);
        if (s == 17) { group_hot(1); group_gather(c, 1); }
        if (s == 20 || s == 21) group_multiply(1, 0, s - 20);
        if (s == 22) { group_hot(0); group_pack(1); }
        if (s == 25 || s == 26) group_multiply(0, 1, s - 25);
        if (s == 27) group_hot(1);
        if (s == 30 || s == 31) group_multiply(1, 1, s - 30);
        if (s & 8) {                                        // next chunk's x: pieces 0, 1 behind 8..15, pieces 2, 3 behind 24..31
          const int i = (s >> 4) * 2 + ((s >> 2) & 1);
          store_x_word(c + 1, i, s & 3);
          if ((s & 3) == 3) load_x(min(s < 16 ? c + 1 : c + 2, nchunks - 1), i ^ 2);
        }
      } else {
        if (s == 12) group_gather(c, 0);
        if (s == 15) group_pack(0);
        if (s == 16) group_gather(c, 1);
        if (s == 17) group_hot(0);
        if (s == 19) group_pack(1);
        if (s >= 20 && s < 24) group_multiply(0, s & 1, (s >> 1) & 1);
        if (s == 24) group_hot(1);
        if (s >= 28) group_multiply(1, s & 1, (s >> 1) & 1);
        if (s == 16) clip_x(c + 1);
        if (s >= 16) {
          store_x_word(c + 1, (s - 16) >> 2, s & 3);
          if ((s & 3) == 3) load_x(min(c + 2, nchunks - 1), (s - 16) >> 2);
        }
      }
      __builtin_amdgcn_sched_barrier(0);
    };
    if constexpr (GROUP_SCALE) {
      // Groups of 128 = one chunk: the products with the integer codes are summed for one block of rows of W at a time,
      // and the sums take the group's scale in fp32.
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        float16_t part[2];
#pragma unroll
        for (int step = 0; step < 8; ++step) {
#pragma unroll
          for (int i = 0; i < 2; ++i) {
            float16_t zero;
#pragma unroll
            for (int r = 0; r < 16; ++r) zero[r] = 0.0f;
            part[i] = Frag<DT>::mfma(a[step & 1][i], __builtin_bit_cast(frag_t, b[step & 1][0]), step == 0 ? zero : part[i]);
            if (j == 0 || step < 7) read_a(c, (step + 1) & 7, i);
            if (step < 7) dequant(step + 1, j, i); else dequant(8, j ^ 1, i);
            if ((step & 3) == 2 && i == 1) load_q(c + 1, step >> 2, j);
            behind(16 * j + 2 * step + i);
          }
        }
        const float scale = (float)__builtin_bit_cast(_Float16, (uint16_t)sc[0][j]);
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
          for (int r = 0; r < 16; ++r) acc[i][j][r] = fmaf(part[i][r], scale, acc[i][j][r]);
        // the sums are done before the next ones begin: there are no registers for a third set
        asm volatile("" : "+v"(acc[0][j]), "+v"(acc[1][j]), "+v"(b[0][0]));
        load_group_scale(c + 1, j);
        __builtin_amdgcn_sched_barrier(0);
      }
    } else {
#pragma unroll
      for (int step = 0; step < 8; ++step) {
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          const int i = u & 1, j = u >> 1;
          acc[i][j] = Frag<DT>::mfma(a[step & 1][i], __builtin_bit_cast(frag_t, b[step & 1][j]), acc[i][j]);
          if (step < 7 && u < 2) read_a(c, step + 1, u);
          // next step's weights: block 0 behind the first two instructions, block 1 behind the others
          dequant(step + 1, u >> 1, u & 1);
          if ((step & 3) == 2 && (u & 1)) load_q(c + 1, step >> 2, u >> 1);        // the tile's last word has been taken
          behind(4 * step + u);
        }
      }
    }
    for (uint32_t g0 = j_lo + 16u; g0 < j_hi; g0 += 16u) group_all(c, g0, j_hi);
    j_lo = j_hi;
    j_hi = j_next;
    __syncthreads();                                        // next chunk's x complete, this one's no longer read
  }

  // ---- epilogue: register r of block (i, j) holds token row 32 i + 8 (r/4) + 4 (lane/32) + r%4, column 32 j + lane%32 of
  //      the wave.  The bf16 target tile is copied to the place of x with coalesced loads first ----
  const FwdParams pe = cold();
  const bool staged = ((pe.N & 7) == 0) && ((reinterpret_cast<uintptr_t>(pe.target) & 15) == 0);
  if (staged) {
    constexpr int CPR = OP_BN / 8, ROWS_PER_PASS = 64 * OP_WAVES / CPR, PASSES = OP_BM / ROWS_PER_PASS, BATCH = 4;
    static_assert(PASSES % BATCH == 0, "whole batches");
    const int cc = tid % CPR, r0 = tid / CPR;
    const int ncl = min(n0 + 8 * cc, pe.N - 8);
#pragma unroll
    for (int bt = 0; bt < PASSES; bt += BATCH) {
      u32x4 t[BATCH];
#pragma unroll
      for (int i = 0; i < BATCH; ++i) {
        const int m = min(m0 + r0 + ROWS_PER_PASS * (bt + i), pe.M - 1);
        t[i] = *reinterpret_cast<global_u32x4>(pe.target + (size_t)m * pe.N + ncl);
      }
#pragma unroll
      for (int i = 0; i < BATCH; ++i)
        *reinterpret_cast<u32x4*>(smem + (r0 + ROWS_PER_PASS * (bt + i)) * OP_TROW + 16 * cc) = t[i];
    }
    __syncthreads();
  }
  const float eps = pe.signed_eps;
  const int ml0 = 4 * half, nl0 = wave * 64 + l31;
  const uint8_t* const trow = smem + ml0 * OP_TROW + nl0 * 2;
  // Without y: with d = D - t the losses are sum d^2 +- 2 eps sum d Z + eps^2 sum Z^2, and their difference, which g
  // is made of, is summed as such instead of being left over from two nearly equal sums.  Squares and products are exact and
  // are added one by one in fp64 (as in the few-token kernels; sixteen at a time in fp32
  // first is no faster: four Llama blocks at 128 tokens 305 against 306 us per step, one block at 4096 on request 2037 against 2041).
  double loss_plus = 0.0, loss_minus = 0.0, sum_dd = 0.0, sum_dz = 0.0, sum_zz = 0.0;
  uint8_t* const special = smem + OnePassLds::RING;         // AGAIN: token rows that are left out
  auto finish = [&](auto full_tag, auto staged_tag, auto again_tag) {
    constexpr bool FULL = decltype(full_tag)::value, STAGED = decltype(staged_tag)::value, AGAIN = decltype(again_tag)::value;
    const uint32_t base = (uint32_t)(m0 + ml0) * (uint32_t)pe.N + (uint32_t)(n0 + nl0);   // M * N < 2^32 checked on the host
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int j = 0; j < 2; ++j) {
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const int dm = 32 * i + 8 * (r >> 2) + (r & 3), dn = 32 * j;
          if ((FULL || (m0 + ml0 + dm < pe.M && n0 + nl0 + dn < pe.N)) && !(AGAIN && special[ml0 + dm])) {
            const uint32_t off = base + (uint32_t)dm * (uint32_t)pe.N + (uint32_t)dn;
            uint32_t tb;
            if (STAGED) tb = *reinterpret_cast<const uint16_t*>(trow + dm * OP_TROW + dn * 2);
            else tb = pe.target[off];
            const float t = __uint_as_float(tb << 16);
            if (STORE_Y || AGAIN) {                         // as mse_kernel: differences and squares in fp64
              const float ez = eps * accz[i][j][r], yp = acc[i][j][r] + ez, ym = acc[i][j][r] - ez;
              if (!AGAIN) pe.y[off] = ym;
              const double dp = (double)yp - (double)t, dmn = (double)ym - (double)t;
              loss_plus = fma(dp, dp, loss_plus);
              loss_minus = fma(dmn, dmn, loss_minus);
            } else {
              const double d = (double)(acc[i][j][r] - t), z = (double)accz[i][j][r];
              sum_dd = fma(d, d, sum_dd);
              sum_dz = fma(d, z, sum_dz);
              sum_zz = fma(z, z, sum_zz);
            }
          }
        }
      }
  };
  using T = std::true_type;
  using F = std::false_type;
  {
    const bool full = m0 + OP_BM <= pe.M && n0 + OP_BN <= pe.N;
    if (full && staged) finish(T{}, T{}, F{});
    else if (staged) finish(F{}, T{}, F{});
    else finish(F{}, F{}, F{});
  }
  if (!STORE_Y) {
    const double even = fma((double)eps * (double)eps, sum_zz, sum_dd), odd = 2.0 * (double)eps * sum_dz;
    loss_plus = even + odd;
    loss_minus = even - odd;
  }
  __shared__ double wave_part[2][OP_WAVES];
  double tile_plus, tile_minus;                             // of the whole workgroup, in every thread
  auto sum_waves = [&]() {
    loss_plus = wave_sum(loss_plus);
    loss_minus = wave_sum(loss_minus);
    if (lane == 0) { wave_part[0][wave] = loss_plus; wave_part[1][wave] = loss_minus; }
    __syncthreads();
    tile_plus = 0.0; tile_minus = 0.0;
#pragma unroll
    for (int i = 0; i < OP_WAVES; ++i) { tile_plus += wave_part[0][i]; tile_minus += wave_part[1][i]; }
  };
  sum_waves();
  if (!(__builtin_isfinite(tile_plus) && __builtin_isfinite(tile_minus))) {
    // Outputs that are not finite.  The squares are added one by one this time (D = inf and Z = 0 have no product); token
    // rows with an infinite or NaN activation are left out and evaluated by their definition, thread = column.
    __syncthreads();
    for (int i = 0; i < OP_BM / OP_WAVES; ++i) {
      const int row = OP_BM / OP_WAVES * wave + i;
      bool bad = false;
      for (int k = 8 * lane; m0 + row < pe.M && k < K; k += 8 * 64) {
        const u32x4 u = *reinterpret_cast<global_u32x4>(pe.x + (size_t)(m0 + row) * K + k);
        for (int w = 0; w < 4; ++w) bad = bad || (u[w] & 0x7F80u) == 0x7F80u || (u[w] & 0x7F800000u) == 0x7F800000u;
      }
      const bool any = __any(bad);
      if (lane == 0) special[row] = any ? 1 : 0;
    }
    __syncthreads();
    loss_plus = 0.0; loss_minus = 0.0;
    finish(F{}, F{}, T{});
    const WeightSource source = {pe.qweight, pe.scales, nullptr, pe.tile_ptr, pe.sp_idx, pe.sp_val, K, gshift, pe.nnz, pe.nnz_base, pe.seed, pe.step};
    for (int row = 0; row < OP_BM; ++row) {
      if (!special[row] || n0 + tid >= pe.N) continue;
      const uint32_t n = (uint32_t)(n0 + tid), off = (uint32_t)(m0 + row) * (uint32_t)pe.N + n;
      const global_u16 x = pe.x + (size_t)(m0 + row) * K;
      float yp = 0.0f, ym = 0.0f;
      nonfinite_output<DT>(source, x, n, eps, yp);
      nonfinite_output<DT>(source, x, n, -eps, ym);
      if (STORE_Y) pe.y[off] = ym;
      const double t = (double)__uint_as_float((uint32_t)pe.target[off] << 16), dp = (double)yp - t, dmn = (double)ym - t;
      loss_plus = fma(dp, dp, loss_plus);
      loss_minus = fma(dmn, dmn, loss_minus);
    }
    sum_waves();
  }
  if (tid == 0) {
    pe.partials[bm * pe.grid_n + bn] = tile_plus * pe.loss_scale;
    pe.partials_minus[bm * pe.grid_n + bn] = tile_minus * pe.loss_scale;
  }
}

// Which forms of the body a kernel holds: the launches over layers of one kind, i.e. almost all of them, take a kernel with
// that one alone.
constexpr int kNoGroups128 = 0, kAllGroups128 = 1, kSomeGroups128 = 2;

// Every layer of a step in one grid: the table (see forward_table) holds one entry per layer, ordered by first_block (a multiple of 8).
template <int DT, bool STORE_Y, int GROUPS, bool SPARSE>
__global__ void __launch_bounds__(64 * OP_WAVES, 2) onepass_table_kernel(const FwdParams* table, int n_entries, InlineForwards) {
  constexpr int W = (int)(sizeof(FwdParams) / 4), FB = (int)(offsetof(FwdParams, first_block) / 4);
  const table_words tab = forward_table(table);
  int first = 0, last = n_entries - 1;                      // last entry whose first_block <= blockIdx.x
  while (first < last) {
    const int mid = (first + last + 1) >> 1;
    if ((int)tab[mid * W + FB] <= (int)blockIdx.x) first = mid; else last = mid - 1;
  }
  const FwdParams p = read_entry(tab + first * W);
  const int bid = (int)blockIdx.x - p.first_block;
  if (bid >= p.grid_m * p.grid_n) return;
  if constexpr (GROUPS == kAllGroups128) onepass_body<DT, STORE_Y, true, SPARSE>(p, bid, tab + first * W);
  else if constexpr (GROUPS == kNoGroups128) onepass_body<DT, STORE_Y, false, SPARSE>(p, bid, tab + first * W);
  else if (p.group_shift == 7) onepass_body<DT, STORE_Y, true, SPARSE>(p, bid, tab + first * W);
  else onepass_body<DT, STORE_Y, false, SPARSE>(p, bid, tab + first * W);
}

// One layer, its descriptor in the kernel arguments.
template <int DT, int GROUPS, bool SPARSE>
__global__ void __launch_bounds__(64 * OP_WAVES, 2) onepass_kernel(FwdParams p) {
  onepass_body<DT, false, GROUPS == kAllGroups128, SPARSE>(p, (int)blockIdx.x, nullptr);
}

// ---- host side -----------------------------------------------------------------------------

template <typename Kernel, typename... Args>
static int launch(Kernel kern, std::atomic<uint64_t>& lds_limit_set, int64_t blocks, hipStream_t stream, Args... args) {
  int rc = set_lds_limit_once(lds_limit_set, (const void*)kern, OnePassLds::BYTES);
  if (rc != SZO_OK) return rc;
  rc = timing_begin(stream);
  if (rc != SZO_OK) return rc;
  kern<<<(unsigned)blocks, 64 * OP_WAVES, OnePassLds::BYTES, stream>>>(args...);
  SZO_LAUNCH_CHECK();
  return timing_end(stream);
}
template <int DT, bool STORE_Y, int GROUPS, bool SPARSE>
static int launch_table(const ForwardTableArgs& t, int64_t blocks, hipStream_t stream) {
  static std::atomic<uint64_t> lds_limit_set{0};             // per instantiation
  return launch(onepass_table_kernel<DT, STORE_Y, GROUPS, SPARSE>, lds_limit_set, blocks, stream, t.table, t.n_entries, t.inl);
}
template <bool STORE_Y, bool SPARSE>
static int launch_table(bool bf16, int groups, const ForwardTableArgs& t, int64_t blocks, hipStream_t stream) {
  if (bf16) return launch_table<SZO_TILE_BF16, STORE_Y, kNoGroups128, SPARSE>(t, blocks, stream);
  if (groups == kNoGroups128) return launch_table<SZO_TILE_F16, STORE_Y, kNoGroups128, SPARSE>(t, blocks, stream);
  if (groups == kAllGroups128) return launch_table<SZO_TILE_F16, STORE_Y, kAllGroups128, SPARSE>(t, blocks, stream);
  return launch_table<SZO_TILE_F16, STORE_Y, kSomeGroups128, false>(t, blocks, stream);
}
template <int DT, int GROUPS, bool SPARSE>
static int launch_one(const FwdParams& p, hipStream_t stream) {
  static std::atomic<uint64_t> lds_limit_set{0};
  return launch(onepass_kernel<DT, GROUPS, SPARSE>, lds_limit_set, (int64_t)p.grid_m * p.grid_n, stream, p);
}
template <bool SPARSE>
static int launch_one(const szo_linear_desc* d, const FwdParams& p, hipStream_t stream) {
  if (d->tile_dtype == SZO_TILE_BF16) return launch_one<SZO_TILE_BF16, kNoGroups128, SPARSE>(p, stream);
  return d->group == 128 ? launch_one<SZO_TILE_F16, kAllGroups128, SPARSE>(p, stream) : launch_one<SZO_TILE_F16, kNoGroups128, SPARSE>(p, stream);
}

// Whether a launch of `wgs` workgroups takes the SPARSE form: the gathers that it saves against the branch in its schedule, which
// costs more where no second workgroup shares the CU (two do from 512 on).  us per call, all sixteen slots gathered -> SPARSE, at
// a density of 0.01 / 0.05 / 0.1 / 0.2 / 0.3 %: one Llama block at 4096 tokens on request 2012 / 2037 / 2068 / 2316 / 2505 -> 1954 / 1996 /
// 2033 / 2327 / 2535, at 300 tokens 182 / 181 / 186 / 204 / 226 -> 176 / 175 / 182 / 206 / 229, sixteen OPT blocks at 64 tokens 602 / 610 / 617 /
// 690 / 760 -> 587 / 590 / 612 / 704 / 770; one 4096 x 4096 layer at 600 tokens (160 workgroups) 65.1 / 65.2 / 67.1 / 80.2 / 88.6 -> 64.6 /
// 64.9 / 68.9 / 84.0 / 92.4, with groups of 64 63.5 / 62.8 / 65.1 / 77.2 / 84.4 -> 62.2 / 61.3 / 66.4 / 80.7 / 88.2; one Llama block with outputs
// at one token (172) at 0.05 / 0.07 / 0.13 / 0.3 % 146 / 146 / 155 / 199 -> 147 / 149 / 163 / 210.  Without the scale in fp32
// there is less to gain at 0.1 % (eight OPT blocks with the bf16 tile at 64 tokens 363 -> 361, one Llama block with groups of 64 at 300 188 ->
// 185) and masks with rows full of entries lose (half of them in 1 % of the rows: two OPT blocks with the bf16 tile at 128 tokens 302 -> 310,
// one with groups of 64 and outputs at 300 273 -> 282; in fp32 two Llama blocks at 2048 2179 -> 2152): the lower line there too,
// and where the longest K outlasts the launch's work spread over the chip (one OPT block with outputs at 300 tokens and 0.1 % 234 -> 239).
constexpr double kSparseEntries = 0.0012, kSparseEntriesAlone = 0.00075;
static bool sparse_launch(double entries, double weights, int64_t wgs, double wg_k, int64_t longest_k, bool group_scale) {
  return entries <= (wgs >= 512 && 1.5 * wg_k >= 512.0 * (double)longest_k && group_scale ? kSparseEntries : kSparseEntriesAlone) * weights;
}

int64_t onepass_tiles(const szo_linear_desc* d) {
  return ((d->M + OP_BM - 1) / OP_BM) * ((d->N + OP_BN - 1) / OP_BN);
}

static int g_force_onepass = 0;                             // testing hook: 1 = wherever the kernel can, -1 = never
void onepass_force(int how) { g_force_onepass = how; }

// Whether a step takes this kernel.  `few`: the few-token path would take the step otherwise; `asked_for`: the caller
// wants one dense pass (SZO_STEP_ONE_DENSE_PASS).  Measured at a density of 0.1 % unless said otherwise, us per step,
// other path -> this one:
//  * against the few-token path: more than 32 tokens and 512 workgroups, two per CU.  Four Llama blocks at 32 / 48 / 64 /
//    128 tokens (700 .. 1400 workgroups) 159 / 232 / 241 / 517 -> 189 / 192 / 193 / 346; one Mistral block at 128 / 192
//    tokens (416 / 624) 153 / 256 -> 204 / 214; 32 OPT blocks at 64 / 224 tokens 1531 / 5697 -> 1241 / 4334.
//    Not up to 64 tokens where the longest K (12 us per 1024 columns here, 7 there) outlasts everything else: four OPT
//    blocks at 64 tokens 214 -> 241.  Where the few-token path has only its split kernel (bf16 tile, K an odd multiple of
//    64): four Llama blocks with the bf16 tile at 17 / 64 / 100 tokens 264 / 500 / 713 -> 218 / 220 / 393; there, and against
//    the 128-row tiles that such layers run on otherwise, both paths are estimated from sizes and density (fitted with
//    split_rounded_us): one OPT block at 128 tokens and 0.1 / 0.7 / 1 %, tiles -> this one 379 / 437 / 463 -> 253 / 473 / 568.
//    Beyond 128 tokens, where that path takes a layer of up to 2304 workgroups, too: 11008 x 4160 with groups of 64 at 200 tokens 77 -> 60,
//    2080 x 448 at 905 30 -> 19, 4590 x 1024 with the bf16 tile at 491 42 -> 32, the other way 3360 x 4288 with it at 535
//    83 against 90, 710 x 4032 at 2009 60 against 80.
//  * asked for at more tokens than the few-token path takes by itself, against its slices: from 160 workgroups on (110
//    with smaller groups, whose slices are slower).  A 2048 x 12288 layer at 512 tokens (64 of them) 91 -> 154, a 4096 x 16384
//    layer at 512 / 700 (128 / 176) 187 / 240 -> 210 / 214.
//    Without slices (bf16 tile, K an odd multiple of 64): wherever it has 32 workgroups and the tiles would run layer by layer,
//    and against a grouped launch, which is slower with that tile, up to 1.75 / 4: two OPT blocks at 224 tokens and 0.4 %
//    636 -> 400, four at 512 tokens and 1 % 1654 -> 2179.
//  * against the tiled kernel, which computes both forwards: the two differ by what a row of tiles
//    costs: a unit of 64 token rows here takes 1 + 108 rho
//    (rho = share of sensitive weights; one Llama block at 2048 tokens, rho = 0.0001 / 0.001 / 0.002 / 0.004 / 0.006:
//    1459 / 1450 / 1448 / 1464 / 1479 -> 1070 / 1079 / 1216 / 1419 / 1662), one of a 256-row tile 1.42 / 4, padding
//    included.  Steps of a handful of workgroups gain nothing: they keep the tiled kernel.
//    Beyond 512 tokens the chip is at its power limit, where masks with rows full of entries and the bf16 tile cost more: one
//    Llama block at 4096 tokens on request, rho = 0.0001 / 0.001 / 0.002 / 0.004: 2759 / 2762 / 2780 / 2832 -> 2058 / 2114 / 2386 / 2864,
//    half the entries in 1 % of the rows at 0.001 / 0.002: 2760 / 2797 -> 2195 / 2489, bf16 tile 2830 -> 2386 at 0.001, 2894 -> 3076
//    at 0.004.
//    Without being asked up to 2048 tokens, or while the tiled launch has eight rounds of workgroups at most: there the last
//    rows of tiles, the last round and the launches per layer weigh as much as the second product.  One Llama block at 520 /
//    1000 / 2048 tokens 582 / 809 / 1416 -> 326 / 548 / 1064; single layers at 600 / 2048 / 8192 tokens: 4096 x 4096 122 / 175 / 462 -> 67 / 101 /
//    352, 1024 x 1024 45 / 41 / 58 -> 19 / 24 / 40, 1024 x 16384 433 / 427 / 672 -> 98 / 180 / 359.  Larger steps keep two
//    products unless asked, up to 4096 tiles of 256 x 256: their losses are the single-layer calls' up to the order of the partial sums.
//    Beyond that they are the tiled kernel's with one dense product (four Llama blocks at 4096 tokens here / there 8100 / 6570, a Mistral
//    block at 8192 4358 / 3420), which also takes steps of this kernel from 512 of those tiles on where this one rounds
//    the weights as well (shared_pays in szo_gemm.hip).  Tiles are counted over the step, so the same layers in smaller
//    steps may fall on the other side of the line, where losses and g differ by the roundings that szo.h describes.
//  * with the outputs written (flags = 0) the other path is two tiled launches and two passes over y per layer: one Llama
//    block at 1 / 256 / 1024 tokens 1044 / 1063 / 1508 -> 150 / 189 / 621; rho = 0.01, 1024 tokens: 1836 -> 1128.
static bool worth_it(const szo_linear_desc* descs, int n, bool few, bool asked_for, bool store_y, bool separate) {
  int64_t wgs = 0, tiles = 0, most_tokens = 0;
  double weights = 0.0, entries = 0.0, here = 0.0, tiled = 0.0, wg_k = 0.0, longest_k = 0.0;
  bool stream = true, groups_of_128 = true, bf16 = false;
  for (int i = 0; i < n; ++i) {
    const szo_linear_desc* d = &descs[i];
    if (d->M == 0 || d->N == 0) continue;
    const double size = (double)d->N * (double)d->K;
    wgs += onepass_tiles(d);
    tiles += ((d->M + 255) / 256) * ((d->N + 127) / 128);
    wg_k += (double)onepass_tiles(d) * (double)d->K;
    longest_k = std::max(longest_k, (double)d->K);
    most_tokens = std::max<int64_t>(most_tokens, d->M);
    weights += size;
    entries += (double)d->nnz;
    here += size * (double)((d->M + 63) / 64);
    tiled += size * (double)((d->M + 255) / 256) * 4.0;
    stream = stream && d->K % 128 == 0 && d->tile_dtype == SZO_TILE_F16;
    groups_of_128 = groups_of_128 && d->group == 128;
    bf16 = bf16 || d->tile_dtype == SZO_TILE_BF16;
  }
  const double rho = entries / weights;
  if (store_y) return wgs >= 4 && rho <= 0.015;
  if (asked_for && stream && !few) return wgs >= (groups_of_128 ? 160 : 110);
  const bool rounded_many = few && !stream && most_tokens > 128;         // the split kernel against this one, both estimated
  if (separate && few && !rounded_many) return false;
  if (!(asked_for && !stream)) {
    if (few && !rounded_many && (wgs < 512 ? stream || most_tokens <= 64 || wgs < 256 : most_tokens <= (stream ? 32 : 16))) return false;
    if (few && stream) return most_tokens > 64 || 205.0 * longest_k <= wg_k;
    if ((!few || rounded_many) && wgs < (most_tokens <= 128 ? 256 : 32)) return false;
  }
  if (!stream && (few || most_tokens <= 128)) {
    // both in units of 1024 columns; beyond 128 tokens fitted again: the launch is shorter there, the walk longer
    const double fixed = rounded_many ? 17.0 : 26.6, walk = !rounded_many ? 9.3 : bf16 ? 13.0 : 10.0;
    auto estimate = [&](double k, double work) {
      return fixed + 3.5 * k + std::max(walk * k * (1.0 + 176.0 * rho), 0.0221 * work * (1.0 + 42.0 * rho));
    };
    double us = estimate(longest_k / 1024.0, wg_k / 1024.0);
    if (rounded_many && separate) {
      us = 0.0;
      for (int i = 0; i < n; ++i)
        if (descs[i].M > 0 && descs[i].N > 0) us += estimate((double)descs[i].K / 1024.0, (double)onepass_tiles(&descs[i]) * (double)descs[i].K / 1024.0);
    }
    if (us >= small_m_rounded_us(descs, n, few, separate)) return false;
    if (few && !rounded_many) return true;
  }
  // asked for in a step too small for a grouped tiled launch (384 tiles of 256 x 128): the tiles would run layer by layer and sign
  if (asked_for && tiles < 384) return wgs >= 32;
  if (!asked_for && most_tokens > 2048 && tiles > 2048) return false;
  const double line = asked_for ? 1.75 : most_tokens <= 512 ? 1.42 : stream ? 1.34 : 1.22;
  return (1.0 + 108.0 * rho) * here < line * tiled;
}

// The outputs are written by concurrent workgroups: layers must not share them (a caller that only wants the losses may
// hand out one buffer for the whole stack).
static bool outputs_overlap(const szo_linear_desc* descs, int n) {
  static thread_local std::vector<std::pair<uintptr_t, uintptr_t>> spans;
  spans.clear();
  for (int i = 0; i < n; ++i) {
    const szo_linear_desc* d = &descs[i];
    if (d->M == 0 || d->N == 0) continue;
    spans.push_back({(uintptr_t)d->y, (uintptr_t)d->y + sizeof(float) * (size_t)d->M * (size_t)d->N});
  }
  std::sort(spans.begin(), spans.end());
  for (size_t i = 1; i < spans.size(); ++i)
    if (spans[i].first < spans[i - 1].second) return true;
  return false;
}

// Loss partials per sign of the step if it takes this kernel, 0 if not.
int64_t onepass_partials(const szo_linear_desc* descs, int n, bool few, bool asked_for, bool store_y, bool separate) {
  if (g_force_onepass < 0) return 0;
  int64_t T = 0;
  const szo_linear_desc* any = nullptr;
  for (int i = 0; i < n; ++i) {
    const szo_linear_desc* d = &descs[i];
    if (d->M == 0 || d->N == 0) continue;
    if (d->format != SZO_FORMAT_UNIFORM || d->x_minus || d->K >= (1 << 23)) return 0;
    if (any && d->tile_dtype != any->tile_dtype) return 0;
    any = d;
    T += onepass_tiles(d);
  }
  if (T == 0 || (g_force_onepass == 0 && !worth_it(descs, n, few, asked_for, store_y, separate))) return 0;
  return store_y && outputs_overlap(descs, n) ? 0 : T;
}

static int fill_tiled(FwdParams& p, const szo_linear_desc* d, uint64_t seed, uint64_t step, float eps, double* plus, double* minus) {
  const int rc = fill_params(p, d, seed, step, +1, eps, plus, 1.0 / ((double)d->M * (double)d->N));
  p.partials_minus = (global_f64_out)minus;
  p.grid_m = (int)((d->M + OP_BM - 1) / OP_BM);
  p.grid_n = (int)((d->N + OP_BN - 1) / OP_BN);
  return rc;
}

int onepass_one(const szo_linear_desc* d, uint64_t seed, uint64_t step, float eps, double* plus, double* minus, hipStream_t stream) {
  FwdParams p;
  const int rc = fill_tiled(p, d, seed, step, eps, plus, minus);
  if (rc != SZO_OK) return rc;
  if (onepass_tiles(d) > 0x7FFFFFFF) return SZO_EUNSUPPORTED;
  return sparse_launch((double)d->nnz, (double)d->N * (double)d->K, onepass_tiles(d), (double)onepass_tiles(d) * (double)d->K, d->K,
                       d->tile_dtype == SZO_TILE_F16 && d->group == 128) ? launch_one<true>(d, p, stream) : launch_one<false>(d, p, stream);
}

int onepass_forwards(const szo_linear_desc* descs, int n, uint64_t seed, uint64_t step, float eps, bool few, bool asked_for,
                     bool store_y, void* table_dev, double* partials, int64_t* partials_per_sign, hipStream_t stream) {
  const int64_t T = onepass_partials(descs, n, few, asked_for, store_y, false);
  if (T == 0 || 2 * T > kMaxLossPartials) return SZO_EUNSUPPORTED;
  static thread_local std::vector<int> order;
  order.clear();
  for (int i = 0; i < n; ++i)
    if (descs[i].M > 0 && descs[i].N > 0) order.push_back(i);
  if (sizeof(FwdParams) * order.size() > kTableBytesPerMatrix * (size_t)kMaxStepMatrices) return SZO_EUNSUPPORTED;
  // longest K first: the last workgroups to start are the shortest
  std::stable_sort(order.begin(), order.end(), [&](int a, int b) { return descs[a].K > descs[b].K; });
  static thread_local std::vector<FwdParams> table;
  table.clear();
  int64_t first_block = 0, offset = 0;
  double entries = 0.0, weights = 0.0, wg_k = 0.0;
  for (int i : order) {
    const szo_linear_desc* d = &descs[i];
    entries += (double)d->nnz;
    weights += (double)d->N * (double)d->K;
    wg_k += (double)onepass_tiles(d) * (double)d->K;
    FwdParams p;
    const int rc = fill_tiled(p, d, seed, step, eps, partials + offset, partials + T + offset);
    if (rc != SZO_OK) return rc;
    p.first_block = (int)first_block;
    table.push_back(p);
    first_block += (onepass_tiles(d) + 7) & ~(int64_t)7;
    if (first_block > 0x7FFFFFFF) return SZO_EUNSUPPORTED;
    offset += onepass_tiles(d);
  }
  static thread_local ForwardTableArgs t;
  const int rc = place_table(table.data(), table.size(), table_dev, stream, t);
  if (rc != SZO_OK) return rc;
  *partials_per_sign = T;
  const int e = (int)table.size(), with = (int)std::count_if(table.begin(), table.end(), [](const FwdParams& p) { return p.group_shift == 7; });
  const int groups = with == e ? kAllGroups128 : with == 0 ? kNoGroups128 : kSomeGroups128;
  const bool bf16 = descs[order[0]].tile_dtype == SZO_TILE_BF16;
  if (sparse_launch(entries, weights, T, wg_k, descs[order[0]].K, !bf16 && groups == kAllGroups128))
    return store_y ? launch_table<true, true>(bf16, groups, t, first_block, stream) : launch_table<false, true>(bf16, groups, t, first_block, stream);
  return store_y ? launch_table<true, false>(bf16, groups, t, first_block, stream) : launch_table<false, false>(bf16, groups, t, first_block, stream);
}

}  // namespace szo
