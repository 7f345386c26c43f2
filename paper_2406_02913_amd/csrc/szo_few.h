// Shared by the kernels of the few-token path (szo_smallm.hip, szo_split.hip): the table entry that describes a
// matrix, the launch arguments, and the register-level dequantisation of 4-bit codes into matrix operands.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <cstddef>
#include "szo_internal.h"
#include "szo_rng.h"

namespace szo {

typedef _Float16 half2_t __attribute__((ext_vector_type(2)));
typedef _Float16 half4_t __attribute__((ext_vector_type(4)));
typedef _Float16 half8_t __attribute__((ext_vector_type(8)));
typedef float float4_t __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef unsigned short u16x2 __attribute__((ext_vector_type(2)));

constexpr int SM_ROWS = 16;             // token rows of the MFMA (M padded up to this)
constexpr int SM_PLAIN = 0, SM_FAST = 1, SM_LUT = 2;        // how the codes are dequantised, see small_m_kernel

struct SmallMat {
  const uint16_t* x;        // bf16 [M,K]
  const uint16_t* x2;       // bf16 [M,K] or null: the -eps forward's activations where they differ (DUAL kernels)
  const uint8_t* qweight;   // [N,K/2]
  const uint16_t* scales;   // fp16 [N,K/group]
  const uint32_t* tile_ptr;
  const uint32_t* sp_idx;
  float* sp_val;
  const uint16_t* target;   // bf16 [M,N]   (loss mode)
  float* y;                 // fp32 [M,N]   (store_sign != 0)
  uint64_t nnz_base;
  double loss_scale;
  int N, K;
  int M;                    // token rows of this entry (<= 16 or <= 32, by instantiation): longer matrices are split into slices
  uint32_t nnz;
  int group_shift;
  uint32_t div_mul;
  int div_shift;
  int first_block;          // workgroups of earlier matrices in this launch
  int partial_base;         // index of this matrix's first loss partial
  int64_t first_quad;       // threads of earlier matrices in the grouped update (one per Philox counter = 4 entries,
                            // rounded up to whole waves of 64 per matrix)
};

static_assert(sizeof(SmallMat) <= kTableBytesPerMatrix, "table entries must fit the workspace's table area");

// Launches over a handful of matrices carry their table in the kernel arguments (read by scalar loads like the rest of
// them) instead of staging it in device memory: one launch and one event record less per step.
static_assert(kInlineMats * sizeof(SmallMat) <= 2048, "kernel arguments are limited to 4 KB");

struct SmallArgs {
  const SmallMat* table;    // device table of n_mats matrices, or null: they are in `inl`
  SmallMat inl[kInlineMats];
  int n_mats;
  uint32_t part_shifts;     // split kernel, 4 bits per matrix of `inl`: its bands are cut into 1 << these workgroups (staged tables: 0)
  int few_rows;             // split kernel: no matrix of the launch has more than four token rows
  int slices;               // slices of token rows per strip in this launch (the longest matrix's count)
  int stream_once;          // host's choice: load the codes as a non-temporal stream (see small_m_kernel, ONCE)
  int store_sign;           // which forward's outputs are written to y (+1, -1), 0: neither
  int loss_mode;            // 1: write loss partials for both signs
  uint64_t seed, step;
  float eps;                // perturbation scale of the "+" forward (the "-" forward uses -eps)
  double* partial_plus;     // [total workgroups]
  double* partial_minus;
};

__device__ __forceinline__ uint32_t sm_fast_div(uint32_t v, uint32_t mul, int shift) {
  const uint32_t t = __umulhi(mul, v);
  return (t + ((v - t) >> 1)) >> shift;
}

// (a & mask) | bits: one v_and_or_b32 when `bits` is in a register.  Plain C on purpose.  As inline assembly
// the instruction is opaque to the compiler's hazard handling, which keeps two wait states between a vector
// instruction that writes a register and a matrix instruction that reads it: here the result IS a matrix
// operand, and with the assembly form sequences with a single wait state were generated (harmless while
// other waves share the SIMD and issue in between, wrong products for a wave that has the SIMD to itself).
__device__ __forceinline__ uint32_t sm_and_or(uint32_t a, uint32_t mask, uint32_t bits_vgpr) {
  return (a & mask) | bits_vgpr;
}

// 8 codes -> 8 fp16 values in the order (0,4)(1,5)(2,6)(3,7).
// RAW: 1024+c for even positions and 64+c for odd ones (the caller removes the constants);
// otherwise (c - 8) times the group scale.
template <bool RAW>
__device__ __forceinline__ half8_t sm_dequant_word(uint32_t q, uint32_t magic_lo, uint32_t magic_hi, half2_t s2) {
  const uint32_t q8 = q >> 8;
  half2_t h0 = __builtin_bit_cast(half2_t, sm_and_or(q, 0x000F000Fu, magic_lo));
  half2_t h1 = __builtin_bit_cast(half2_t, sm_and_or(q, 0x00F000F0u, magic_hi));
  half2_t h2 = __builtin_bit_cast(half2_t, sm_and_or(q8, 0x000F000Fu, magic_lo));
  half2_t h3 = __builtin_bit_cast(half2_t, sm_and_or(q8, 0x00F000F0u, magic_hi));
  if (!RAW) {
    const half2_t off_lo = {(_Float16)1032.0f, (_Float16)1032.0f}, off_hi = {(_Float16)72.0f, (_Float16)72.0f};
    h0 = (h0 - off_lo) * s2; h1 = (h1 - off_hi) * s2; h2 = (h2 - off_lo) * s2; h3 = (h3 - off_hi) * s2;
  }
  half8_t r;
  r[0] = h0[0]; r[1] = h0[1]; r[2] = h1[0]; r[3] = h1[1];
  r[4] = h2[0]; r[5] = h2[1]; r[6] = h3[0]; r[7] = h3[1];
  return r;
}

// word w of the staged form of 8 bf16 values: (x[w], x[w+4]) as fp16
__device__ __forceinline__ uint32_t sm_stage_x_word(u32x4 u, int w) {
  const uint32_t first = (w < 2) ? u[0] : u[1], second = (w < 2) ? u[2] : u[3];
  float a, b;
  if ((w & 1) == 0) { a = __uint_as_float(first << 16); b = __uint_as_float(second << 16); }
  else              { a = __uint_as_float(first & 0xFFFF0000u); b = __uint_as_float(second & 0xFFFF0000u); }
  auto h = __builtin_amdgcn_cvt_pkrtz(a, b);
  return __builtin_bit_cast(uint32_t, h);
}

// Eight codes of one row -> eight fp16 table values in the order (0,4)(1,5)(2,6)(3,7).  The row's table of 16
// entries is held as four byte planes T = {low bytes of entries 0-7, high bytes of 0-7, low bytes of 8-15,
// high bytes of 8-15}, two registers each: the byte permute looks up four codes at a time by their low
// three bits, and bit 3 picks the plane through a byte mask.
__device__ __forceinline__ half8_t sm_lut_word(uint32_t q, const uint32_t (&T)[8]) {
  const uint32_t sel_e = q & 0x07070707u, sel_o = (q >> 4) & 0x07070707u;         // even codes 0,2,4,6 | odd codes 1,3,5,7
  const uint32_t m_e = __builtin_amdgcn_perm(0u, 0x0000FF00u, (q >> 3) & 0x01010101u);   // 0xFF where the code is >= 8
  const uint32_t m_o = __builtin_amdgcn_perm(0u, 0x0000FF00u, (q >> 7) & 0x01010101u);
  auto pick = [](uint32_t m, uint32_t b, uint32_t a) { return (m & b) | (~m & a); };
  const uint32_t lo_e = pick(m_e, __builtin_amdgcn_perm(T[5], T[4], sel_e), __builtin_amdgcn_perm(T[1], T[0], sel_e));
  const uint32_t hi_e = pick(m_e, __builtin_amdgcn_perm(T[7], T[6], sel_e), __builtin_amdgcn_perm(T[3], T[2], sel_e));
  const uint32_t lo_o = pick(m_o, __builtin_amdgcn_perm(T[5], T[4], sel_o), __builtin_amdgcn_perm(T[1], T[0], sel_o));
  const uint32_t hi_o = pick(m_o, __builtin_amdgcn_perm(T[7], T[6], sel_o), __builtin_amdgcn_perm(T[3], T[2], sel_o));
  const u32x4 w = {__builtin_amdgcn_perm(hi_e, lo_e, 0x06020400u),      // codes 0, 4
                   __builtin_amdgcn_perm(hi_o, lo_o, 0x06020400u),      // codes 1, 5
                   __builtin_amdgcn_perm(hi_e, lo_e, 0x07030501u),      // codes 2, 6
                   __builtin_amdgcn_perm(hi_o, lo_o, 0x07030501u)};     // codes 3, 7
  return __builtin_bit_cast(half8_t, w);
}

// Pointers read out of a table are generic to the compiler; say that they are global memory, or every access
// becomes a flat load with conservative waits on both memory counters.
#define SZO_GLOBAL(T, p) ((const T __attribute__((address_space(1)))*)(p))

// Workgroup ids go round-robin over the 8 XCDs, each with its own L2.  Remapped so that eight consecutive units
// (normally of one matrix, which all read the same x) run on one XCD and consecutive groups of eight rotate over
// the XCDs; the ragged tail (< 64 ids) keeps its order.
__device__ __forceinline__ int xcd_unit(int bid, int grid) {
  if (bid < (grid & ~63)) {
    const int xcd = bid & 7, i = bid >> 3;
    bid = (((i >> 3) << 3) + xcd) * 8 + (i & 7);
  }
  return bid;
}

// Table entry of workgroup `unit`: the last matrix whose first_block <= unit.  Read through the constant address
// space (scalar loads: the table is written before the launch and never during it), so that its fields live in
// scalar registers like the kernel arguments do; read through a generic pointer they would occupy ~30 vector
// registers.
typedef const uint32_t __attribute__((address_space(4)))* small_words;
__device__ __forceinline__ small_words small_table(const SmallArgs& a) {
  return a.table ? (small_words)a.table : (small_words)__builtin_amdgcn_kernarg_segment_ptr() + offsetof(SmallArgs, inl) / 4;
}
__device__ __forceinline__ int find_index(small_words tab, int n_mats, int unit) {
  constexpr int W = (int)(sizeof(SmallMat) / 4), FB = (int)(offsetof(SmallMat, first_block) / 4);
  static_assert(sizeof(SmallMat) % 4 == 0 && offsetof(SmallMat, first_block) % 4 == 0, "table entry is read as words");
  int lo = 0, hi = n_mats - 1;
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if ((int)tab[mid * W + FB] <= unit) lo = mid; else hi = mid - 1;
  }
  return lo;
}
__device__ __forceinline__ SmallMat read_matrix(small_words tab, int index) {
  constexpr int W = (int)(sizeof(SmallMat) / 4);
  struct Words { uint32_t w[W]; } raw;
#pragma unroll
  for (int i = 0; i < W; ++i) raw.w[i] = tab[index * W + i];
  return __builtin_bit_cast(SmallMat, raw);
}
__device__ __forceinline__ SmallMat find_matrix(const SmallArgs& a, int unit) {
  const small_words tab = small_table(a);
  return read_matrix(tab, find_index(tab, a.n_mats, unit));
}

// The tables of one row, 16 fp16 entries at p, as the four byte planes that sm_lut_word() reads.
__device__ __forceinline__ void load_lut_planes(const uint16_t __attribute__((address_space(1)))* p, uint32_t (&T)[8]) {
  const auto* lp = reinterpret_cast<const u32x4 __attribute__((address_space(1)))*>(p);
  const u32x4 lo = lp[0], hi = lp[1];                       // entries 0-7 and 8-15, two per word
  T[0] = __builtin_amdgcn_perm(lo[1], lo[0], 0x06040200u); T[1] = __builtin_amdgcn_perm(lo[3], lo[2], 0x06040200u);
  T[2] = __builtin_amdgcn_perm(lo[1], lo[0], 0x07050301u); T[3] = __builtin_amdgcn_perm(lo[3], lo[2], 0x07050301u);
  T[4] = __builtin_amdgcn_perm(hi[1], hi[0], 0x06040200u); T[5] = __builtin_amdgcn_perm(hi[3], hi[2], 0x06040200u);
  T[6] = __builtin_amdgcn_perm(hi[1], hi[0], 0x07050301u); T[7] = __builtin_amdgcn_perm(hi[3], hi[2], 0x07050301u);
}

// One-hot operands of the sparse product: entry i (0..3) of this lane's k-group belongs to row (word & 15) of 16-row
// subtile (word >> 4) & 3.  mlo / mhi hold 0xFFFF in halfword s of the pair iff this lane owns the entry's row in
// subtile s and the entry counts.
__device__ __forceinline__ void one_hot_entry(uint32_t row, int nn, bool counts, uint32_t& mlo, uint32_t& mhi) {
  const bool mine = counts && (row & 15u) == (uint32_t)nn;
  const uint64_t m = (uint64_t)0xFFFFu << (row & 0x30u);    // 16 * subtile
  mlo = mine ? (uint32_t)m : 0u;
  mhi = mine ? (uint32_t)(m >> 32) : 0u;
}

// One launch of the split kernel (szo_split.hip): a workgroup per band or part of one and slice of 16 token rows.
struct SplitLaunch {
  int mode;                 // SM_*
  bool dual, bf16, tile_round;
  bool one;                 // only the "+" forward is wanted (used by tile_round)
  int subs;                 // most subtiles of a workgroup: 4 >> the smallest part shift of the launch
  int waves, workgroups;
  int64_t longest_k;
};
int split_launch(const SplitLaunch& l, const SmallArgs& a, hipStream_t stream);

}  // namespace szo
