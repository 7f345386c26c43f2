// Behind the main loop of a 256 x 256 tile that has computed D = x (dq + v)^T: the sensitive product Z = x z^T of the same outputs, and
// the losses of both forwards, y(+-) = D +- eps Z (Section 3.4; both forwards of a layer see the same x).
//
// The entries of a tile are few (at 0.1 %, four per column of outputs), but D fills half of the registers and Z has as many sums, so Z is
// not carried through the main loop.  Afterwards a wave keeps Z of 64 x 64 of its 128 x 64 outputs at a time and multiplies its band's
// entries thirty-two at a time: their columns of x, and a one-hot operand (z at [row of W][slot]).  The columns come from a copy of x in
// which 64 tokens of one column are 128 contiguous bytes in the tile's 16-bit type (transpose_kernel), so that a tile fetches only the
// columns that its entries want, 0.5 MB at 0.1 % and K = 4096 where the whole of x is 2 MB; they go from memory to LDS without passing
// through registers and are turned into the matrix operand by the transposing LDS read.  Every wave has buffers of its own and none
// waits for another.
//
// Two Llama blocks at 4096 tokens, 0.1 %, us: two full products in dual-sign tiles 5130, this 3290, of which the dense product and the
// losses are 2730 and the copies 203 (576 MB read and written at 5.7 TB/s).  A group takes its entries from LDS while the one before is
// multiplied, and the one-hot operand is read in two halves, which leaves the main loop all of its registers: 3350 without.  The same with x streamed through LDS again, 2 MB per
// tile, and its columns gathered there 3960; with Z carried through the main loop of 256 x 128 tiles 4220.
//
// A buffer holds 32 "rows" (columns of x, or rows of targets) of 128 bytes; their 16-byte piece c stands in slot c ^ swizzle(row), so that the eight
// rows that half a wave reads side by side lie in different banks.  (A load to LDS puts 64 lanes side by side; the lanes choose what
// they read.)
#pragma once
#include <type_traits>
#include "szo_nonfinite.h"
#include "szo_rng.h"
#include "szo_tile.h"

namespace szo {

constexpr int SH_WIN = 480;                                 // sensitive entries held per wave, a multiple of 32
constexpr int SH_BUF = 32 * 128;                            // bytes of one group of columns; three of them per wave
struct SharedLds {                                          // byte offsets, per wave and of the workgroup
  static constexpr int HOT = 3 * SH_BUF, WIN = HOT + 64 * 64, WAVE = WIN + 8 * SH_WIN;
  static constexpr int SINK = 8 * WAVE, SPECIAL = SINK + 8 * 64, BYTES = SPECIAL + 256;
};
static_assert(SH_WIN % 32 == 0 && SharedLds::BYTES + 512 <= 160 * 1024, "one workgroup per CU");

// A copy of activations with 64 tokens of a column side by side: [block of 64 rows][K][64 rows], in the tile's type, rows past M zero.
// Each wave turns 64 x 64 values through LDS of its own.  Bound by memory: one read and one write of x.
struct TransposeItem { const uint16_t* x; uint16_t* out; int M, K; uint32_t first; };        // first: of its blocks of 64 x 64
struct TransposeArgs { TransposeItem item[8]; int n; uint32_t blocks; };
typedef __attribute__((address_space(3))) uint8_t* lds_bytes_t;
typedef short lds_short4 __attribute__((ext_vector_type(4)));
__device__ __forceinline__ uint64_t read_transposed(lds_bytes_t at) {  // lane l of sixteen: values l%16 of the four 32-byte rows that lanes 4 t + .. point into
  return __builtin_bit_cast(uint64_t, __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) lds_short4*)at));
}
template <int DT>
__global__ void __launch_bounds__(256) transpose_kernel(TransposeArgs t) {
  __shared__ alignas(16) uint8_t tile[4][64 * 128];
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6), n = lane & 15, kg = lane >> 4;
  const uint32_t block = 4u * blockIdx.x + (uint32_t)wave;
  if (block >= t.blocks) return;                            // waves share nothing
  int which = 0;
  for (int i = 1; i < t.n; ++i) which = block >= t.item[i].first ? i : which;
  const TransposeItem it = t.item[which];
  const int ktiles = it.K / 64, mb = (int)((block - it.first) / (uint32_t)ktiles), kt = (int)((block - it.first) % (uint32_t)ktiles);
  const int m0 = 64 * mb;
  u32x4 v[8];
#pragma unroll
  for (int i = 0; i < 8; ++i)
    v[i] = *reinterpret_cast<global_u32x4>((global_u16)it.x + (size_t)min(m0 + 8 * i + (lane >> 3), it.M - 1) * it.K + 64 * kt + 8 * (lane & 7));
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    const bool inside = m0 + 8 * i + (lane >> 3) < it.M;
    u32x4 w;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const uint32_t u = inside ? v[i][e] : 0u;
      if (DT == SZO_TILE_F16) w[e] = __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_pkrtz(__uint_as_float(u << 16), __uint_as_float(u & 0xFFFF0000u)));
      else w[e] = u;
    }
    const int slot = (lane & 7) ^ (2 * ((lane >> 4) & 1)) ^ (4 * (i & 1));
    *reinterpret_cast<u32x4*>(&tile[wave][(8 * i + (lane >> 3)) * 128 + 16 * slot]) = w;
  }
  asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");        // visible to the wave's other lanes
  const lds_bytes_t from = (lds_bytes_t)&tile[wave][(8 * kg + (n >> 2)) * 128 + 16 * ((n >> 1) & 1) + 8 * (n & 1)];
  const uint32_t swizzle = 32u * (uint32_t)((n >> 3) | ((kg & 1) << 1));
  uint8_t* const out = reinterpret_cast<uint8_t*>(it.out) + ((size_t)mb * it.K + 64 * kt) * 128;
#pragma unroll
  for (int c = 0; c < 4; ++c)                               // sixteen columns
#pragma unroll
    for (int q = 0; q < 2; ++q) {                           // 32 rows
      const lds_bytes_t at = from + 32 * q * 128 + ((32u * (uint32_t)c) ^ swizzle);
      const uint64_t lo = read_transposed(at), hi = read_transposed(at + 4 * 128);
      *reinterpret_cast<u32x4*>(out + (16 * c + n) * 128 + 64 * q + 16 * kg) = u32x4{(uint32_t)lo, (uint32_t)(lo >> 32), (uint32_t)hi, (uint32_t)(hi >> 32)};
    }
}

template <int DT, bool FP64_SUMS, typename ReadEntry>
__device__ __forceinline__ void shared_tail(float4_t (&acc)[8][4], const ReadEntry& cold, const int bm, const int bn, uint8_t* const smem) {
  typedef typename Frag<DT>::type operand_t;
  const FwdParams p = cold();
  int tid = threadIdx.x;
  asm volatile("" : "+v"(tid));                             // what is formed of it is formed here, not held through the main loop
  const int lane = tid & 63, n = lane & 15, kg = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), wm = wave >> 2, wn = wave & 3;
  const int m0 = bm * 256, n0 = bn * 256, K = p.K;
  const int band = n0 / 64 + wn;
  const bool band_ok = band < p.bands && p.nnz > 0;
  const float eps = p.signed_eps;
  uint8_t* const mine = smem + wave * SharedLds::WAVE;
  const lds_bytes_t mine_lds = (lds_bytes_t)mine;

  // ---- 32 rows of 128 bytes to LDS.  Addresses out of the buffer's bounds (rows past M, no such block of rows) read as zero.  In
  //      assembly: behind the compiler's own form it waits for all of them at every LDS read.  Five wait states: a vector instruction, a
  //      reload of a spilled scalar, may have written the descriptor just before ----
  typedef uint32_t rsrc_t __attribute__((ext_vector_type(4)));
  auto buffer = [](uint64_t base, uint32_t bytes) { return rsrc_t{(uint32_t)base, (uint32_t)(base >> 32) & 0xFFFFu, bytes, 0x00027000u}; };
  auto load_rows = [&](rsrc_t rsrc, const uint32_t (&at)[4], uint32_t buf) {
    const uint32_t lds = (uint32_t)(uintptr_t)mine_lds + buf;
    // m0 is no register that values are allocated to, which the compiler warns of; named all the same, so that none of its own
    // settings of m0 is taken to live on behind these
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_mov_b32 m0, %0\n\ts_nop 4\n\t"
                 "buffer_load_dwordx4 %1, %5, 0 offen lds\n\ts_add_u32 m0, m0, 0x400\n\ts_nop 0\n\t"
                 "buffer_load_dwordx4 %2, %5, 0 offen lds\n\ts_add_u32 m0, m0, 0x400\n\ts_nop 0\n\t"
                 "buffer_load_dwordx4 %3, %5, 0 offen lds\n\ts_add_u32 m0, m0, 0x400\n\ts_nop 0\n\t"
                 "buffer_load_dwordx4 %4, %5, 0 offen lds" ::
                 "s"(lds), "v"(at[0]), "v"(at[1]), "v"(at[2]), "v"(at[3]), "s"(rsrc) : "memory", "scc", "m0");
#pragma clang diagnostic pop
  };
  const uint32_t piece = 16u * (uint32_t)((lane & 7) ^ (2 * ((lane >> 4) & 1)));       // row 8 i + lane / 8: ^ 64 for odd i
  const uint32_t block_bytes = 128u * (uint32_t)K;          // K < 2^21
  const int row_blocks = (p.M + 63) / 64;
  const bool staged = ((p.N & 7) == 0) && ((reinterpret_cast<uintptr_t>(p.target) & 15) == 0) && p.N < (1 << 22);

  // ---- sensitive entries: byte offset of the column in a block of x, and z << 16 | byte offset of the row of W in the one-hot operand ----
  uint32_t* const win = reinterpret_cast<uint32_t*>(mine + SharedLds::WIN);
  uint8_t* const hot = mine + SharedLds::HOT;               // [64 rows of W][32 slots]
  uint8_t* const sink = smem + SharedLds::SINK + wave * 64 + 4 * n;
  const table_words bounds = (table_words)(uintptr_t)(p.tile_ptr + (band_ok ? (size_t)band * (size_t)p.ktiles : 0));     // scalar loads
  const uint32_t lo = band_ok ? bounds[0] : 0u, hi = band_ok ? bounds[p.ktiles] : 0u, begin = lo & ~3u;
  const int groups = lo < hi ? (int)((hi - begin + 31u) / 32u) : 0;
  uint32_t win_lo = 0, win_hi = 0;
  auto fill = [&](uint32_t s) {                             // entries [s, s + SH_WIN) of the matrix, s a multiple of 4 below nnz
#pragma unroll 1
    for (uint32_t part = 0; part < 2; ++part) {
      const uint32_t o = 256u * part + 4u * (uint32_t)lane, j = s + o;
      u32x4 column = {0u, 0u, 0u, 0u}, word = {0u, 0u, 0u, 0u};
      if (s + 256u * part < hi) {
        float z[4] = {0.0f, 0.0f, 0.0f, 0.0f};
        if (eps != 0.0f) zbar_quad((p.nnz_base + j) >> 2, p.seed, p.step, z);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const uint32_t idx = p.sp_idx[min(j + e, p.nnz - 1u)];      // clamped; entries past the end are never consumed
          const uint32_t row = fast_div(idx, p.div_mul, p.div_shift);
          uint16_t zb;
          Frag<DT>::store(&zb, z[e]);
          column[e] = (idx - row * (uint32_t)K) << 7;
          word[e] = ((uint32_t)zb << 16) | (((row - (uint32_t)(band * 64)) & 63u) << 6);
        }
      }
      if (o < (uint32_t)SH_WIN) {
        *reinterpret_cast<u32x4*>(win + o) = column;
        *reinterpret_cast<u32x4*>(win + SH_WIN + o) = word;
      }
    }
    win_lo = s;
    win_hi = s + (uint32_t)SH_WIN;
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");      // the window is visible to the wave's other lanes
  };

  // ---- what goes through the three buffers, in order: for each half of the wave's rows its groups of entries, then its targets in two
  //      parts.  Three are under way at any time ----
  int next_half = 0, next_item = 0, ahead = 0;              // ahead: loads under way
  uint32_t next_buf = 0, word[4] = {1u, 1u, 1u, 1u};        // the slots' entries of the groups under way and of the next; odd: none
  uint32_t column[4];                                       // of the next group: where this lane's pieces stand in a block of x
  uint8_t* hot_at = sink;                                   // where this lane's last entry stands
  auto look_ahead = [&]() {                                 // reads the next group's entries; anything if it is no group
    const bool group = next_half < 2 && next_item < groups;
    const uint32_t g0 = begin + 32u * (uint32_t)next_item;
    if (group && (g0 < win_lo || g0 + 32u > win_hi)) fill(g0);
    const uint32_t* const at = win + (group ? g0 - win_lo : 0u);
#pragma unroll
    for (int i = 0; i < 4; ++i) column[i] = at[8 * i + (lane >> 3)];
    const uint32_t j = g0 + (uint32_t)lane, w = at[SH_WIN + (lane & 31)];
    word[3] = group && lane < 32 && j >= lo && j < hi ? w : 1u;
  };
  auto issue = [&](bool targets) {
    word[0] = word[1];
    word[1] = word[2];
    word[2] = word[3];
    __builtin_amdgcn_s_waitcnt(0xC07F);                     // lgkmcnt(0): the buffer has been read
    if (next_half < 2) {
      uint32_t at[4];
      rsrc_t rsrc;
      if (next_item < groups) {
        const int block = 4 * bm + 2 * wm + next_half;
#pragma unroll
        for (int i = 0; i < 4; ++i) at[i] = column[i] + (piece ^ (64u * (uint32_t)(i & 1)));
        rsrc = buffer((uint64_t)(uintptr_t)p.x_minus + (uint64_t)block * block_bytes, block < row_blocks ? block_bytes : 0u);
      } else {
        const int part = next_item - groups;
        const uint32_t row = (uint32_t)(128 * wm + 64 * next_half + 32 * part + (lane >> 3)), pitch = 2u * (uint32_t)p.N;
#pragma unroll
        for (int i = 0; i < 4; ++i) at[i] = (row + 8u * (uint32_t)i) * pitch + 2u * (uint32_t)(n0 + 64 * wn) + (piece ^ (64u * (uint32_t)(i & 1)));
        rsrc = buffer((uint64_t)(uintptr_t)(p.target + (size_t)m0 * p.N), staged && targets ? (uint32_t)min(p.M - m0, 256) * pitch : 0u);
      }
      load_rows(rsrc, at, next_buf);
      ++ahead;
      next_buf = next_buf == 2 * SH_BUF ? 0u : next_buf + SH_BUF;
      if (++next_item == groups + 2) { next_item = 0; ++next_half; }
    }
  };
  // For the groups after this: the one-hot operand of the next that is multiplied, the entries of the next that is fetched.
  auto prepare = [&]() {
    asm volatile("" ::: "memory");                          // (other types than what is read before and behind: order)
    *reinterpret_cast<uint16_t*>(hot_at) = 0;
    hot_at = (word[0] & 1u) ? sink : hot + (word[0] & 0xFC0u) + 2 * lane;
    *reinterpret_cast<uint16_t*>(hot_at) = (uint16_t)(word[0] >> 16);
    look_ahead();
  };
  uint32_t buf = 0;                                         // of the oldest load under way
  auto arrived = [&]() {
    if (ahead == 3) asm volatile("s_waitcnt vmcnt(8)" ::: "memory");
    else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  };
  auto consumed = [&](bool targets) {                       // everything read from it, the reads perhaps under way
    --ahead;
    buf = buf == 2 * SH_BUF ? 0u : buf + SH_BUF;
    issue(targets);
  };

  float4_t accz[4][4];
  const uint32_t from = (uint32_t)(8 * kg + (n >> 2)) * 128u + 16u * (uint32_t)((n >> 1) & 1) + 8u * (uint32_t)(n & 1);
  const uint32_t swizzle = 32u * (uint32_t)((n >> 3) | ((kg & 1) << 1));
  auto multiply = [&](bool targets) {
    arrived();
    u32x4 a[4], b[2];
    auto read_b = [&](int j) { return *reinterpret_cast<const u32x4*>(hot + (16 * j + n) * 64 + 16 * kg); };
    auto product = [&](int j) {
#pragma unroll
      for (int i = 0; i < 4; ++i) accz[i][j] = Frag<DT>::mfma16(__builtin_bit_cast(operand_t, a[i]), __builtin_bit_cast(operand_t, b[j & 1]), accz[i][j]);
    };
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const lds_bytes_t at = mine_lds + buf + from + ((32u * (uint32_t)i) ^ swizzle);
      const uint64_t first = read_transposed(at), second = read_transposed(at + 4 * 128);
      a[i] = u32x4{(uint32_t)first, (uint32_t)(first >> 32), (uint32_t)second, (uint32_t)(second >> 32)};
    }
    b[0] = read_b(0);
    consumed(targets);
    b[1] = read_b(1);
    product(0);
    b[0] = read_b(2);
    product(1);
    b[1] = read_b(3);
    product(2);
    prepare();
    product(3);
  };

  // With d = D - t the losses are sum d^2 +- 2 eps sum d Z + eps^2 sum Z^2; the difference of the losses, which g is made of, is summed as
  // such.  FP64_SUMS: squares and products, exact there, are added one by one in fp64, as in the one-dense-pass kernel; otherwise
  // sixteen at a time in fp32 and those sums in fp64, as in the dual-sign tiles: 1.7 us less of 151 per tile at K = 4096 (32 Llama blocks
  // at 4096 tokens 59.7 -> 59.1 ms), a few 1e-9 of the losses.
  double loss_plus = 0.0, loss_minus = 0.0, sum_dd = 0.0, sum_dz = 0.0, sum_zz = 0.0;
  uint8_t* const special = smem + SharedLds::SPECIAL;       // AGAIN: token rows that are left out
  auto finish = [&](int half, auto part_tag, auto full_tag, auto staged_tag, auto again_tag) {
    constexpr bool FULL = decltype(full_tag)::value, STAGED = decltype(staged_tag)::value, AGAIN = decltype(again_tag)::value;
    constexpr int PART = decltype(part_tag)::value;         // 32 rows
    const int ml = 128 * wm + 64 * half + 4 * kg, nl = 64 * wn + n;
    const uint32_t base = (uint32_t)(m0 + ml) * (uint32_t)p.N + (uint32_t)(n0 + nl);         // M * N < 2^32 checked on the host
    const lds_bytes_t t0 = mine_lds + buf + (uint32_t)(4 * kg + (n >> 2)) * 128u + 16u * (uint32_t)((n >> 1) & 1) + 8u * (uint32_t)(n & 1);
    const uint32_t t_swizzle = 32u * (uint32_t)((n >> 3) | ((kg >> 1) << 1));
#pragma unroll
    for (int i = 2 * PART; i < 2 * PART + 2; ++i) {
      float dd = 0.0f, dz = 0.0f, zz = 0.0f;
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const uint64_t four = STAGED ? read_transposed(t0 + 16 * (i & 1) * 128 + ((32u * (uint32_t)j) ^ t_swizzle)) : 0;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int dm = 16 * i + r, dn = 16 * j;
          if ((FULL || (m0 + ml + dm < p.M && n0 + nl + dn < p.N)) && !(AGAIN && special[ml + dm])) {
            uint32_t tb;
            if (STAGED) tb = (uint32_t)(four >> (16 * r)) & 0xFFFFu;
            else tb = p.target[base + (uint32_t)dm * (uint32_t)p.N + (uint32_t)dn];
            const float t = __uint_as_float(tb << 16), df = half ? acc[4 + i][j][r] : acc[i][j][r], zf = accz[i][j][r];
            if (AGAIN) {
              const float ez = eps * zf;
              const double dp = (double)(df + ez) - (double)t, dmn = (double)(df - ez) - (double)t;
              loss_plus = fma(dp, dp, loss_plus);
              loss_minus = fma(dmn, dmn, loss_minus);
            } else if (FP64_SUMS) {
              const double d = (double)(df - t), z = (double)zf;
              sum_dd = fma(d, d, sum_dd);
              sum_dz = fma(d, z, sum_dz);
              sum_zz = fma(z, z, sum_zz);
            } else {
              const float d = df - t;
              dd = fmaf(d, d, dd);
              dz = fmaf(d, zf, dz);
              zz = fmaf(zf, zf, zz);
            }
          }
        }
      }
      if (!AGAIN && !FP64_SUMS) {
        sum_dd += (double)dd;
        sum_dz += (double)dz;
        sum_zz += (double)zz;
      }
    }
  };
  using T = std::true_type;
  using F = std::false_type;
  const bool full = m0 + 256 <= p.M && n0 + 256 <= p.N;

  // Z of one half and its share of the losses.
  auto one_half = [&](auto half, auto again_tag) {
    constexpr bool AGAIN = decltype(again_tag)::value;
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int j = 0; j < 4; ++j) accz[i][j] = float4_t{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll 1
    for (int g = 0; g < groups; ++g) multiply(!AGAIN);
    auto part = [&](auto which) {
      arrived();
      if (AGAIN) finish(half, which, F{}, F{}, T{});
      else if (full && staged) finish(half, which, T{}, T{}, F{});
      else if (staged) finish(half, which, F{}, T{}, F{});
      else finish(half, which, F{}, F{}, F{});
      consumed(!AGAIN);
      prepare();
    };
    part(std::integral_constant<int, 0>{});
    part(std::integral_constant<int, 1>{});
  };
  auto begin_loads = [&](bool targets) {
    next_half = 0;
    look_ahead();
    for (int i = 0; i < 3; ++i) { issue(targets); prepare(); }
  };
  __syncthreads();                                          // every wave is done with the main loop's buffers
#pragma unroll
  for (int i = 0; i < 4; ++i) *reinterpret_cast<u32x4*>(hot + 1024 * i + 16 * lane) = u32x4{0u, 0u, 0u, 0u};
  begin_loads(true);
  one_half(std::integral_constant<int, 0>{}, F{});
  one_half(std::integral_constant<int, 1>{}, F{});
  {
    const double even = fma((double)eps * (double)eps, sum_zz, sum_dd), odd = 2.0 * (double)eps * sum_dz;
    loss_plus = even + odd;
    loss_minus = even - odd;
  }
  __shared__ double wave_part[2][8];
  double tile_plus, tile_minus;                             // of the whole workgroup, in every thread
  auto sum_waves = [&]() {
    loss_plus = wave_sum(loss_plus);
    loss_minus = wave_sum(loss_minus);
    if (lane == 0) { wave_part[0][wave] = loss_plus; wave_part[1][wave] = loss_minus; }
    __syncthreads();
    tile_plus = 0.0; tile_minus = 0.0;
#pragma unroll
    for (int i = 0; i < 8; ++i) { tile_plus += wave_part[0][i]; tile_minus += wave_part[1][i]; }
  };
  sum_waves();
  if (!(__builtin_isfinite(tile_plus) && __builtin_isfinite(tile_minus))) {
    // Outputs that are not finite: the squares one by one (D = inf and Z = 0 have no product), token rows with an infinite or NaN activation
    // by their definition, thread = column.
    __syncthreads();
    for (int row = wave; row < 256; row += 8) {
      bool bad = false;
      for (int k = 8 * lane; m0 + row < p.M && k < K; k += 8 * 64) {
        const u32x4 u = *reinterpret_cast<global_u32x4>(p.x + (size_t)(m0 + row) * K + k);
        for (int w = 0; w < 4; ++w) bad = bad || (u[w] & 0x7F80u) == 0x7F80u || (u[w] & 0x7F800000u) == 0x7F800000u;
      }
      const bool any = __any(bad);
      if (lane == 0) special[row] = any ? 1 : 0;
    }
    __syncthreads();                                        // `special` is there
    begin_loads(false);
    loss_plus = 0.0; loss_minus = 0.0;
#pragma unroll 1
    for (int half = 0; half < 2; ++half) one_half(half, T{});
    const WeightSource source = {p.qweight, p.scales, nullptr, p.tile_ptr, p.sp_idx, p.sp_val, K, p.group_shift, p.nnz, p.nnz_base, p.seed, p.step};
    for (int row = tid >> 8; row < 256; row += 2) {
      const int col = n0 + (tid & 255);
      if (!special[row] || col >= p.N) continue;
      const global_u16 x = p.x + (size_t)(m0 + row) * K;
      float yp = 0.0f, ym = 0.0f;
      nonfinite_output<DT>(source, x, (uint32_t)col, eps, yp);
      nonfinite_output<DT>(source, x, (uint32_t)col, -eps, ym);
      const double t = (double)__uint_as_float((uint32_t)p.target[(size_t)(m0 + row) * p.N + col] << 16), dp = (double)yp - t, dmn = (double)ym - t;
      loss_plus = fma(dp, dp, loss_plus);
      loss_minus = fma(dmn, dmn, loss_minus);
    }
    sum_waves();
  }
  if (tid == 0) {
    p.partials[bm * p.grid_n + bn] = tile_plus * p.loss_scale;
    p.partials_minus[bm * p.grid_n + bn] = tile_minus * p.loss_scale;
  }
}

}  // namespace szo
