// Shared by the translation units of libszo: error bookkeeping and the layout of the
// loss workspace.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <atomic>
#include "szo.h"

namespace szo {

extern thread_local int g_last_hip_error;

inline int hip_failed(hipError_t e) {
  if (e == hipSuccess) return 0;
  g_last_hip_error = (int)e;
  return 1;
}

#define SZO_HIP(expr) do { if (::szo::hip_failed((expr))) return SZO_ELAUNCH; } while (0)
#define SZO_LAUNCH_CHECK() SZO_HIP(hipGetLastError())

// Raises a kernel's dynamic LDS limit once per device (`done` holds one bit per device id); safe to
// call from several host threads.
inline int set_lds_limit_once(std::atomic<uint64_t>& done, const void* fn, size_t bytes) {
  int dev = 0;
  SZO_HIP(hipGetDevice(&dev));
  const uint64_t bit = 1ull << (dev & 63);
  if (done.load(std::memory_order_acquire) & bit) return SZO_OK;
  SZO_HIP(hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes));
  done.fetch_or(bit, std::memory_order_release);
  return SZO_OK;
}

// Loss workspace: 64 reserved bytes followed by one fp64 partial per workgroup.  A kernel launched behind the one
// that wrote them adds the partials in index order, which makes the sum independent of scheduling.
constexpr int kMaxLossPartials = 1 << 21;       // 16 MiB: a 32-block 7B stack at 4096 tokens has 2 x 340 000 dual-sign tiles
constexpr size_t kWorkspaceHeader = 64;
constexpr int kMaxStepMatrices = 4096;            // descriptor table of the few-token step
constexpr size_t kTableBytesPerMatrix = 144;
constexpr size_t kWorkspaceTableOffset = kWorkspaceHeader + sizeof(double) * (size_t)kMaxLossPartials;
// Copies of activations, column by column, for the sensitive products of large steps: a step goes in launches of as many layers as fit.
constexpr size_t kWorkspaceCopyOffset = kWorkspaceTableOffset + kTableBytesPerMatrix * (size_t)kMaxStepMatrices;
// Steps that write none are content with the part before it.
constexpr size_t kSmallWorkspaceBytes = kWorkspaceCopyOffset;
constexpr size_t kCopyAreaBytes = (size_t)1 << 30;
constexpr size_t kWorkspaceBytes = kWorkspaceCopyOffset + kCopyAreaBytes + 128;

// loss_acc[0] += scale * sum of partials[0..count) in a fixed order (one workgroup).
int reduce_partials(const double* partials, int count, double scale, double* loss_acc, hipStream_t stream);
// scalars[0] = sum partials[0..count), scalars[1] = sum partials[count..2*count), scalars[2] = SPSA g.
int reduce_step(const double* partials, int count, float eps, double* scalars, hipStream_t stream);

// Whether a launch of 128 x 128 tiles, one forward, computes K in two parts side by side (szo_gemm.hip).  While every tile has a CU to itself: a
// workgroup of two parts takes a CU's LDS, where two whole tiles would share it, so from 257 tiles on the parts only take turns.  Both
// parts walk the same number of K steps of 64 columns, at least two; three where the tiles nearly fill the chip, where two gain and lose.
// us of one forward with 0.1 % sensitive, one part -> two: 4096 x 4096 at 460 / 1000 tokens (128 / 256 tiles) 42.3 / 52.9 -> 35.3 / 41.7
// (the first against the few-token path), with 1 % in half of the rows at 450 87.8 -> 53.4, 1024 x 8192 at 3000 99.5 -> 68.8,
// 1024 x 512 at 2000 11.5 -> 9.9, 2000 x 256 at 700 8.5 -> 7.7, the seven layers of a Llama block at 600 506 -> 388.  256 columns: 1536
// rows at 1500 / 1900 tokens (144 / 180 tiles) 8.8 / 9.2 -> 8.2 / 8.6; beyond the line 2077 at 1763 (238) 10.2 -> 10.3, 2048 at 2048 (256)
// 9.3 -> 9.5, 1500 at 1900 9.2 -> 9.1, 3200 at 1000 9.2 -> 8.8, 6400 at 500 9.5 -> 8.8; 2077 x 384 at 1763 11.5 -> 11.2.
constexpr int64_t kTwoPartTiles = 256, kTwoPartColumns = 256;       // most tiles, fewest columns
inline bool tiles_halve_k(int64_t tiles, int64_t K) {
  return tiles <= kTwoPartTiles && K % 128 == 0 && K >= (tiles <= 192 ? kTwoPartColumns : 384);
}

// Few-token path (szo_smallm.hip, szo_split.hip).
// Whether every layer of a launch is taken: few enough tokens to run as slices of 16 or more token rows, or, with
// any_token_count, a shape that the stream kernel takes whatever its number of tokens.  `forwards`: 2 for a step, 1 for the
// single-forward calls (what the tiled kernel would have to do instead).  `separate`: one launch per layer; a step of such
// launches takes no second activation set.
bool small_m_eligible(const szo_linear_desc* descs, int n, bool any_token_count, bool separate, int forwards);
// Whether it takes a single forward (szo_linear_fwd, szo_linear_fwd_mse); `perturbed`: of sign +1 or -1 with eps != 0.
bool small_m_takes_forward(const szo_linear_desc* d, bool perturbed);
// Estimated us of a step's forwards where the stream kernel does not take every layer: on the few-token path (`few`) or in the tiled
// kernel.  Fitted up to 128 tokens and, for single layers, from 129 to 4000.
double small_m_rounded_us(const szo_linear_desc* descs, int n, bool few, bool separate);
// Loss partials per sign of a single-matrix launch, one per workgroup: per strip and slice of the stream kernel, per band or part of
// one and slice of the split kernel.  Callers with little room ask for fewer: as chosen by size (kBandsInParts), bands not cut, or
// the stream kernel where it can.
enum Partials { kBandsInParts, kWholeBands, kStreamKernel };
int64_t small_m_launch_partials(const szo_linear_desc* d, Partials less);
void small_m_force_split(int how);                          // testing hook: 1 = the split kernel always, -1 = only where nothing else can, 0 = choose
void small_m_force_rblocks(int r);                         // testing hook: 0 = choose; 2, 3 = 32 / 48 token rows per pass wherever M > 16
void small_m_force_stream_once(bool on);                    // testing hook: non-temporal code stream in every one-slice launch
size_t small_m_table_bytes(int n);
int small_m_launch_one(const szo_linear_desc* d, uint64_t seed, uint64_t step, float eps, int store_sign, bool loss_mode, bool both_signs,
                       double* partial_plus, double* partial_minus, Partials less, hipStream_t stream);
int small_m_step(const szo_linear_desc* descs, int n, uint64_t seed, uint64_t step, float eps, float lr,
                 void* table_dev, double* partial_plus, int64_t partials_per_sign, double* scalars, bool do_forward,
                 hipStream_t stream);
constexpr int kInlineMats = 8;                              // matrices whose table travels in the kernel arguments

// Many tokens, one dense product per layer (szo_onepass.hip): both forwards of every layer as one launch, the loss fused
// and, with store_y, the -eps outputs written.  SZO_EUNSUPPORTED, with nothing enqueued, when the stack does not qualify.
int onepass_forwards(const szo_linear_desc* descs, int n, uint64_t seed, uint64_t step, float eps, bool few, bool asked_for,
                     bool store_y, void* table_dev, double* partials, int64_t* partials_per_sign, hipStream_t stream);
// The same for callers without a table: how many loss partials per sign the step has if it takes this kernel (0: it does
// not), and one layer's launch.  `separate`: every layer is a launch of its own.
int64_t onepass_partials(const szo_linear_desc* descs, int n, bool few, bool asked_for, bool store_y, bool separate);
int64_t onepass_tiles(const szo_linear_desc* d);            // loss partials per sign of one layer
int onepass_one(const szo_linear_desc* d, uint64_t seed, uint64_t step, float eps, double* plus, double* minus, hipStream_t stream);
void onepass_force(int how);                                // testing hook: 1 = wherever the kernel can, -1 = never, 0 = choose

// Optional kernel timing (szo_kernel_timing): when switched on, every launch of a forward kernel
// (kind 0) or of a sparse update kernel (kind 1) is bracketed by a pair of events on its own stream.
// Both calls are no-ops when timing is off.  Defined in szo_kernels.hip.
int timing_begin(hipStream_t stream, int kind = 0);
int timing_end(hipStream_t stream);

// Copies `bytes` (a multiple of 4) of host data into device memory `dst`, in stream order, without
// blocking the host: the data goes through a ring of eight pinned, device-mapped host buffers per host
// thread (grown on demand with hipHostMalloc, released when the thread ends) and a small copy kernel
// reads it from there.  SZO_EUNSUPPORTED while `stream` is being captured into a graph.  A kernel rather than a
// DMA copy because handing over from the copy engine to the compute queue costs more than reading a
// few tens of KB over the host link.  Defined in szo_kernels.hip.
int stage_table(const void* src, size_t bytes, void* dst, hipStream_t stream);

// True while `stream` is being captured into a HIP graph.
bool stream_is_capturing(hipStream_t stream);

// Sets n 32-bit words to zero with a small kernel (defined in szo_kernels.hip).
int zero_words(void* p, int n, hipStream_t stream);

// Wave-wide sum in a fixed order (64 lanes): halves, then rows of 16, 8, 4, 2, 1 lanes added to each other; result valid in every
// lane.  By lane swaps and row rotations, which stay in registers: the same sums by shuffles are six round trips through LDS, of two
// permutations each, one after the other: 0.3 us at the end of kernels that take five.  (A row rotated by 4, 2 or 1 pairs the lanes that an exclusive or
// would: after each step the sums repeat with that period.)
template <int ROTATE>
__device__ __forceinline__ double add_row_rotated(double v) {
  const uint64_t b = __builtin_bit_cast(uint64_t, v);
  const uint32_t lo = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)b, 0x120 + ROTATE, 0xF, 0xF, false);
  const uint32_t hi = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)(b >> 32), 0x120 + ROTATE, 0xF, 0xF, false);
  return v + __builtin_bit_cast(double, (uint64_t)lo | ((uint64_t)hi << 32));
}
__device__ __forceinline__ double wave_sum(double v) {
#if defined(__HIP_DEVICE_COMPILE__)
  {
    const uint64_t b = __builtin_bit_cast(uint64_t, v);
    const auto lo = __builtin_amdgcn_permlane32_swap((uint32_t)b, (uint32_t)b, false, false);
    const auto hi = __builtin_amdgcn_permlane32_swap((uint32_t)(b >> 32), (uint32_t)(b >> 32), false, false);
    v = __builtin_bit_cast(double, (uint64_t)lo[0] | ((uint64_t)hi[0] << 32)) + __builtin_bit_cast(double, (uint64_t)lo[1] | ((uint64_t)hi[1] << 32));
  }
  {
    const uint64_t b = __builtin_bit_cast(uint64_t, v);
    const auto lo = __builtin_amdgcn_permlane16_swap((uint32_t)b, (uint32_t)b, false, false);
    const auto hi = __builtin_amdgcn_permlane16_swap((uint32_t)(b >> 32), (uint32_t)(b >> 32), false, false);
    v = __builtin_bit_cast(double, (uint64_t)lo[0] | ((uint64_t)hi[0] << 32)) + __builtin_bit_cast(double, (uint64_t)lo[1] | ((uint64_t)hi[1] << 32));
  }
  v = add_row_rotated<8>(v);
  v = add_row_rotated<4>(v);
  v = add_row_rotated<2>(v);
  v = add_row_rotated<1>(v);
#endif
  return v;
}

}  // namespace szo
