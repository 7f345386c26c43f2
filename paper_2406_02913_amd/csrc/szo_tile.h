// Shared by the kernels that stage tiles for the matrix cores: the launch descriptor, the layout of a staged tile in
// LDS, the register-level staging of activations and 4-bit codes, and the map from workgroup ids to output tiles.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <cstddef>
#include <cstring>
#include "szo_internal.h"

namespace szo {

typedef _Float16 half2_t __attribute__((ext_vector_type(2)));
typedef _Float16 half8_t __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef float float2_t __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef float float16_t __attribute__((ext_vector_type(16)));
typedef float float4_t __attribute__((ext_vector_type(4)));

constexpr int BK = 64;                 // K extent of one staged tile = SZO_TILE_COLS
constexpr int kWindow = 256;           // sensitive entries computed per refill of a wave's window

// Device pointers of a descriptor.  In device code they say that they are global memory: a pointer that comes out of a
// table in memory is generic to the compiler, and a generic (flat) load counts on the LDS counter as well, so that every
// wait for an LDS operand also waits for whatever load was issued before it.  Measured on the grouped launches, same machine:
// one Llama block at 4096 tokens 2914 -> 2849 us, eight of them 22.65 -> 22.20 ms, two Mistral blocks at 333 tokens with
// two activation sets 980 -> 935 us.
#ifdef __HIP_DEVICE_COMPILE__
#define SZO_GLOBAL_PTR(T) T __attribute__((address_space(1)))*
#else
#define SZO_GLOBAL_PTR(T) T*
#endif
typedef SZO_GLOBAL_PTR(const uint8_t) global_u8;
typedef SZO_GLOBAL_PTR(const uint16_t) global_u16;
typedef SZO_GLOBAL_PTR(const uint32_t) global_u32;
typedef SZO_GLOBAL_PTR(const float) global_f32;
typedef SZO_GLOBAL_PTR(const u32x4) global_u32x4;
typedef SZO_GLOBAL_PTR(float) global_f32_out;
typedef SZO_GLOBAL_PTR(double) global_f64_out;

struct FwdParams {
  global_u16 x;             // bf16 [M,K]
  global_u8 qweight;        // [N,K/2]
  global_u16 scales;        // fp16 [N,K/group]
  global_u32 tile_ptr;
  global_u32 sp_idx;
  global_f32 sp_val;
  global_f32_out y;         // may be null when the loss is fused
  global_u16 target;        // bf16 [M,N] (fused loss only)
  int M, N, K;
  int group_shift;          // log2(group)
  int ktiles;               // K / 64
  int bands;                // ceil(N / 64)
  int grid_m, grid_n;
  uint32_t nnz;
  uint32_t div_mul;         // exact division of a flat index by K: see fast_div
  int div_shift;
  uint64_t nnz_base, seed, step;
  float signed_eps;         // sign * eps; 0 = no perturbation
  global_f64_out partials;  // fused loss: one scaled partial per workgroup, [grid_m*grid_n]
  double loss_scale;
  int first_block;          // grouped launch: id of this entry's first workgroup (a multiple of 8)
  int pad_;
  global_u16 lut;           // fp16 [N,16], table format only
  // grouped launch: one entry runs BOTH forwards of its matrix; the fields above describe the +eps one
  global_u16 x_minus;       // activations of the -eps forward (= x unless the layer has a second set)
  global_f64_out partials_minus;   // loss partials of the -eps forward
};

// The table of a grouped launch: staged in device memory, or, up to kInlineForwards entries, in the kernel's arguments, where it
// costs no copy kernel in front of the launch.  us per step, staged -> in the arguments: 4096 x 4096 at 200 tokens 37.8 -> 34.6, 2048 x 1024 at
// 500 19.0 -> 16.9, with outputs at 100 67.5 -> 60.5, one Llama block at 256 172 -> 166, one Mistral block with two sets at 333 358 -> 345.
// (A staged launch passes the arguments' table too, unread: whatever the thread's last table was.)
constexpr int kInlineForwards = 16;
struct InlineForwards { FwdParams e[kInlineForwards]; };
struct ForwardTableArgs { const FwdParams* table; int n_entries; InlineForwards inl; };          // as the arguments lie in memory
static_assert(sizeof(ForwardTableArgs) <= 4096 - 256, "kernel arguments are limited to 4 KB, the runtime's own among them");
typedef const uint32_t __attribute__((address_space(4)))* table_words;         // read through scalar loads
__device__ __forceinline__ table_words forward_table(const FwdParams* table) {
  return table ? (table_words)table : (table_words)__builtin_amdgcn_kernarg_segment_ptr() + offsetof(ForwardTableArgs, inl) / 4;
}

// floor(v / d) for 32-bit v with a precomputed multiplier (Granlund-Montgomery, round-up form).
__device__ __forceinline__ uint32_t fast_div(uint32_t v, uint32_t mul, int shift) {
  const uint32_t t = __umulhi(mul, v);
  return (t + ((v - t) >> 1)) >> shift;
}

// Position of column kk (0..63) of tile row r inside the LDS tile, in 16-bit elements.
// Rows are 64 elements (128 bytes), so two rows span the 64 four-byte banks; the eight
// 16-byte chunks of a row are XOR-swizzled with row_swizzle(row), chosen for both ways the tile is
// accessed with 16 bytes per lane.  Reads are served 16 lanes (256 bytes) per cycle: 16 lanes reading the
// same chunk of 16 consecutive rows must touch every bank exactly once, which (row / 2) mod 8 gives.
// Writes are served 8 lanes (128 bytes) per cycle and conflict when two of them fall into the same 16 bytes
// modulo 128, whatever the row's parity (measured: a weight wave writing one chunk of 64 consecutive rows
// took 16 cycles instead of 8 with the (row / 2) swizzle alone, 15 % of all LDS cycles of the kernel);
// the extra (row & 1) * 4 makes 8 consecutive rows distinct as well, and keeps the read property.
// In f16 mode the eight elements of a chunk are stored in the order
// 0,4,1,5,2,6,3,7 -- the order in which two nibbles per 16-bit lane fall out of a packed
// word -- and the activations are stored in the same order, which leaves the dot product
// unchanged.
__device__ __forceinline__ int row_swizzle(int r) { return ((r >> 1) & 7) ^ ((r & 1) << 2); }

template <int DT>
__device__ __forceinline__ int lds_pos(int r, int kk) {
  const int chunk = kk >> 3, w = kk & 7;
  const int p = (DT == SZO_TILE_F16) ? (((w & 3) << 1) | (w >> 2)) : w;
  return r * BK + (((chunk ^ row_swizzle(r)) << 3) | p);
}

__device__ __forceinline__ int chunk_off(int r, int chunk) {   // in 16-bit elements
  return r * BK + ((chunk ^ row_swizzle(r)) << 3);
}

// ---- activations: word w (0..3) of the staged form of one 16-byte chunk of 8 bf16 --------------
// f16 mode pairs elements (0,4) (1,5) (2,6) (3,7); bf16 -> fp32 is a shift and fp32 -> fp16 is
// exact for |x| in [2^-14, 65504] (8-bit significand).
template <int DT>
__device__ __forceinline__ uint32_t stage_x_word(u32x4 u, int w) {
  if (DT == SZO_TILE_BF16) return u[w];
  const uint32_t first = (w < 2) ? u[0] : u[1], second = (w < 2) ? u[2] : u[3];
  float a, b;
  if ((w & 1) == 0) { a = __uint_as_float(first << 16); b = __uint_as_float(second << 16); }
  else              { a = __uint_as_float(first & 0xFFFF0000u); b = __uint_as_float(second & 0xFFFF0000u); }
  auto h = __builtin_amdgcn_cvt_pkrtz(a, b);
  return __builtin_bit_cast(uint32_t, h);
}

// ---- weights: word w (0..3) of the 8 dequantised elements of one 32-bit word of codes ----------
// dq = (code - 8) * scale, one rounding to the tile type.  f16 mode: a nibble in mantissa bits
// 0..3 under exponent pattern 0x6400 reads 1024 + code, one in bits 4..7 under 0x5400 reads
// 64 + code; removing the offset is exact and the product with the fp16 scale is rounded once,
// which is the rounding of the exact (code-8)*scale.  Output pairs are codes (0,4) (1,5) (2,6) (3,7).
// (a & mask) | bits in one VALU instruction, `bits` in a VGPR.  Inline assembly keeps the instruction in
// the slot it is written in (as plain C the tiled step measured 1 % slower).  The compiler's hazard
// handling cannot see into it, which is safe here and only here: the result feeds packed-half arithmetic
// and an LDS store, never a matrix instruction, whose operands all come from LDS reads
// (tests/test_isa_hazards.py checks the generated code for exactly that).
__device__ __forceinline__ uint32_t and_or(uint32_t a, uint32_t mask, uint32_t bits_vgpr) {
  uint32_t r;
  asm("v_and_or_b32 %0, %1, %2, %3" : "=v"(r) : "v"(a), "s"(mask), "v"(bits_vgpr));
  return r;
}

struct DequantConsts { uint32_t magic_lo, magic_hi; };   // 0x64006400 and 0x54005400 held in VGPRs

template <int DT>
__device__ __forceinline__ uint32_t dequant_out(uint32_t q, int w, float scale_f32, half2_t scale_h2,
                                                const DequantConsts& k) {
  if (DT == SZO_TILE_F16) {
    const uint32_t src = (w < 2) ? q : (q >> 8);
    half2_t h;
    if ((w & 1) == 0) {
      h = __builtin_bit_cast(half2_t, and_or(src, 0x000F000Fu, k.magic_lo));
      const half2_t off = {(_Float16)1032.0f, (_Float16)1032.0f};
      h = (h - off) * scale_h2;
    } else {
      h = __builtin_bit_cast(half2_t, and_or(src, 0x00F000F0u, k.magic_hi));
      const half2_t off = {(_Float16)72.0f, (_Float16)72.0f};
      h = (h - off) * scale_h2;
    }
    return __builtin_bit_cast(uint32_t, h);
  } else {
    const float m8s = -8.0f * scale_f32;
    float2_t f = {fmaf((float)((q >> (8 * w)) & 15u), scale_f32, m8s),          // exact in fp32
                  fmaf((float)((q >> (8 * w + 4)) & 15u), scale_f32, m8s)};
    bf16x2_t b = __builtin_convertvector(f, bf16x2_t);                            // round to nearest even
    return __builtin_bit_cast(uint32_t, b);
  }
}

template <int DT> struct Frag;
template <> struct Frag<SZO_TILE_F16> {
  typedef half8_t type;
  static __device__ __forceinline__ float16_t mfma(type a, type b, float16_t c) {
    return __builtin_amdgcn_mfma_f32_32x32x16_f16(a, b, c, 0, 0, 0);
  }
  static __device__ __forceinline__ float4_t mfma16(type a, type b, float4_t c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_f16(a, b, c, 0, 0, 0);
  }
  static __device__ __forceinline__ float load(const uint16_t* p) { return (float)*reinterpret_cast<const _Float16*>(p); }
  static __device__ __forceinline__ void store(uint16_t* p, float v) { *reinterpret_cast<_Float16*>(p) = (_Float16)v; }
};
template <> struct Frag<SZO_TILE_BF16> {
  typedef bf16x8_t type;
  static __device__ __forceinline__ float16_t mfma(type a, type b, float16_t c) {
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
  }
  static __device__ __forceinline__ float4_t mfma16(type a, type b, float4_t c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
  }
  static __device__ __forceinline__ float load(const uint16_t* p) { return __uint_as_float((uint32_t)*p << 16); }
  static __device__ __forceinline__ void store(uint16_t* p, float v) { *reinterpret_cast<__bf16*>(p) = (__bf16)v; }
};

// Workgroup id -> output tile.  Workgroup ids go round-robin over the 8 XCDs, each with its own L2, so
// ids with equal (id % 8) are first made consecutive ("logical" id): the workgroups resident on one XCD
// at a time (32 with the 256x256 tile) are then a run of consecutive logical ids, and logical ids walk
// the tile grid in strips of `strip` row blocks, so that run covers strip x (32 / strip) tiles which
// share `strip` activation strips and 32 / strip weight strips through that L2.  `count` ids in all;
// `bid`'s residue mod 8 is its XCD both in a launch of its own and in a grouped launch (entries start
// at multiples of 8).
__device__ __forceinline__ int logical_block(int bid, int count) {
  const int q = count >> 3, r = count & 7;
  const int xcd = bid & 7, idx = bid >> 3;
  return xcd * q + min(xcd, r) + idx;
}
__device__ __forceinline__ void tile_of_logical(int L, int grid_m, int grid_n, int strip, int& bm, int& bn) {
  const int width = strip * grid_n, g = L / width, first_m = strip * g;
  const int gsize = min(grid_m - first_m, strip), rem = L - g * width;
  bm = first_m + rem % gsize;
  bn = rem / gsize;
}

// Host: where a grouped launch finds its `count` entries: in `inl`, or at table_dev if there are more; whether they are there.
inline bool use_table(const FwdParams* entries, size_t count, const FwdParams* table_dev, ForwardTableArgs& args) {
  args.n_entries = (int)count;
  args.table = count <= (size_t)kInlineForwards ? nullptr : table_dev;
  if (!args.table) memcpy((void*)args.inl.e, entries, count * sizeof(FwdParams));
  return args.table != nullptr;
}
// ... staged at table_dev in that case.
inline int place_table(const FwdParams* entries, size_t count, void* table_dev, hipStream_t stream, ForwardTableArgs& args) {
  return use_table(entries, count, (const FwdParams*)table_dev, args) ? stage_table(entries, sizeof(FwdParams) * count, table_dev, stream) : SZO_OK;
}

// Host: fills the per-layer part of `p` (szo_gemm.hip).
int fill_params(FwdParams& p, const szo_linear_desc* d, uint64_t seed, uint64_t step, int sign, float eps,
                double* partials, double scale);

}  // namespace szo
