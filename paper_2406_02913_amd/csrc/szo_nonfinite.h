// Outputs of token rows that hold an infinite or NaN activation, for the kernels that add the sensitive weights as
// one-hot products of their own: there such an activation also meets zeros that stand for no weight (the other rows of a
// one-hot operand, the zero code under a sensitive weight), and 0 * inf turns outputs into NaN that are infinite by
// y = x (dq + v +- eps z)^T.  A kernel that finds a non-finite output evaluates it again here, one output at a time and
// from the non-finite activations alone: next to them the finite ones add nothing.  Never reached with finite activations.
#pragma once
#include "szo_rng.h"
#include "szo_tile.h"

namespace szo {

struct WeightSource {
  global_u8 qweight;
  global_u16 scales;        // null with tables
  global_u16 lut;           // fp16 [N,16] or null
  global_u32 tile_ptr, sp_idx;
  global_f32 sp_val;
  int K, group_shift;
  uint32_t nnz;
  uint64_t nnz_base, seed, step;
};

// dq + v + signed_eps z of (n, k), rounded as it stands in the tiled kernel's weight tile.
template <int DT>
__device__ inline float weight_at(const WeightSource& s, uint32_t n, uint32_t k, float signed_eps) {
  const uint32_t K = (uint32_t)s.K, band = n >> 6, r = n & 63u;
  const size_t tile = (size_t)band * (K >> 6) + (k >> 6);
  const uint32_t code = ((uint32_t)s.qweight[(tile * 64 + r) * 32 + ((k & 63u) >> 1)] >> (4u * (k & 1u))) & 15u;
  uint16_t w;
  if (s.lut) {
    w = s.lut[(size_t)n * 16 + code];
  } else {
    const uint16_t scale = s.scales[((size_t)band * (K >> s.group_shift) + (k >> s.group_shift)) * 64 + (r & 15u) * 4 + (r >> 4)];
    Frag<DT>::store(&w, ((float)code - 8.0f) * (float)__builtin_bit_cast(_Float16, scale));
  }
  if (s.nnz > 0) {
    for (uint32_t j = s.tile_ptr[tile]; j < s.tile_ptr[tile + 1]; ++j) {
      if (s.sp_idx[j] != n * K + k) continue;
      float z[4] = {0.0f, 0.0f, 0.0f, 0.0f};
      if (signed_eps != 0.0f) zbar_quad((s.nnz_base + j) >> 2, s.seed, s.step, z);
      const float zj = (j & 2u) ? ((j & 1u) ? z[3] : z[2]) : ((j & 1u) ? z[1] : z[0]);
      Frag<DT>::store(&w, Frag<DT>::load(&w) + fmaf(signed_eps, zj, s.sp_val[j]));
    }
  }
  return Frag<DT>::load(&w);
}

// Output n of the token row x [K] (16-byte aligned) if the row holds a non-finite activation; otherwise false and `y` as it was.
template <int DT>
__device__ inline bool nonfinite_output(const WeightSource& s, global_u16 x, uint32_t n, float signed_eps, float& y) {
  bool any = false;
  float sum = 0.0f;
  for (int k0 = 0; k0 < s.K; k0 += 8) {
    const u32x4 u = *reinterpret_cast<global_u32x4>(x + k0);
    for (int e = 0; e < 8; ++e) {
      const uint32_t bits = (u[e >> 1] >> (16 * (e & 1))) & 0xFFFFu;
      if ((bits & 0x7F80u) != 0x7F80u) continue;
      any = true;
      sum = fmaf(__uint_as_float(bits << 16), weight_at<DT>(s, n, (uint32_t)(k0 + e), signed_eps), sum);
    }
  }
  if (any) y = sum;
  return any;
}

}  // namespace szo
