// Perturbed forward of one linear layer (Appendix C.5, "SparseAdd then DenseMM";
// perturbation of Definition 4) as one fused kernel for gfx950:
//
//   4-bit codes --dequantise--> 16-bit tile in LDS  <--scatter--  sp_val[j] + sign*eps*z_j
//   activations (bf16) -------> 16-bit tile in LDS
//   tiles --MFMA 16x16x32--> fp32 accumulators --> y (fp32) and/or sum (y - target)^2 (fp64)
//
// The dense fp weight never exists in memory and the perturbation costs no pass over HBM: it
// is regenerated from (seed, step, entry index) for exactly the entries of the band a wave
// stages.
//
// Work split inside a workgroup.  The first BN/64 waves ("weight waves") each own one 64-row
// band of the weight tile: they load its codes and scales, dequantise them into LDS, and
// scatter the band's sensitive entries on top.  Dense write and sparse overwrite of one LDS
// word are therefore ordered by program order inside one wave and need no barrier.  The other
// waves ("activation waves") convert and stage x.  All waves then run the MFMA loop on the
// staged tile while they stage the next one into the other LDS buffer.
//
// Sensitive entries.  The sparse layout orders entries by (64-row band, 64-column tile), so a
// weight wave consumes its band's entries as one stream while it walks along K.  It computes
// them 256 at a time (one Philox counter = four consecutive entries per lane) into a small
// LDS window holding (tile position, value), and each K step only copies the few entries of
// its tile from the window into the weight tile.
#include <algorithm>
#include <cstddef>
#include <unordered_map>
#include <vector>
#include "szo_internal.h"
#include "szo_rng.h"
#include "szo_shared.h"
#include "szo_tile.h"
#include <mutex>
#include <type_traits>

// Loss partials of szo_zo_step_noalloc: one fp64 value per workgroup and sign, written by the forward
// kernels and summed by reduce_step_kernel.  Lives in the code object, one copy per GPU, for callers
// that cannot allocate a workspace.  Host code never uses this name as an address: it asks the runtime
// for the array's device address once per device (noalloc_partials below).
constexpr int kNoAllocMaxPartials = 1 << 17;                 // 1 MiB per GPU
static __device__ __align__(256) double scratch[kNoAllocMaxPartials];

namespace szo {

// LDS of a tile: two stages of both operands, the weight waves' windows and write sinks.
enum { kNotShared, kShared, kSharedFp64Sums };              // SHARED below
constexpr int tiled_lds_bytes(int bm, int bn) { return 2 * (bm + bn) * BK * (int)sizeof(uint16_t) + (bn / 64) * (kWindow * 6 + 128); }

// Workgroup = WAVES_M x WAVES_N waves; each wave computes (32*WMB) x (32*WNB) outputs.
//
// Schedule of one K step of one wave.  The wave issues SLOTS = 4*WMB*WNB pairs of 16x16x32 MFMAs (or as many 32x32x16).  Its staging
// work for the NEXT tile (8 units per lane: 16-byte chunks of x, or 32-bit words of codes) is
// cut into SLOTS slices of three to four VALU instructions, and one slice is issued behind
// each pair of MFMAs, where it executes in the shadow of the matrix pipeline.  The LDS reads of
// later operands stand between them (see run_tile).  A scheduling fence after every slot keeps
// the compiler from regrouping the slots.  Global loads are in place: as soon as a unit's
// registers have been consumed they are reloaded with the same unit of the tile after next,
// which gives every load one full K step (about a microsecond) to arrive.
// DUAL (grouped launch of a step, loss fused, both forwards read the same activations): the workgroup
// computes BOTH forwards of a tile of BM x BN/2 outputs.  Rows [0, BN/2) of the weight tile in LDS hold
// W + eps z, rows [BN/2, BN) the same rows of W with W - eps z: the codes are loaded and dequantised once
// and written twice, the two copies differ only at the sensitive entries.  Waves of the first half of a
// wave row compute the +eps forward, the others the -eps forward; every MFMA of both forwards is
// executed, only the staging of the weights is shared.  The MFMA loop is the same as without DUAL.
// SHARED (likewise, sparse masks): D of 256 x 256 outputs, without the perturbation, and behind it the sensitive products that both
// forwards add to it (szo_shared.h), the losses summed sixteen at a time in fp32 or one by one in fp64.
//
// KS = 2 (a launch of few 128 x 128 tiles): eight waves, of which the second four compute the second half of the K steps in
// buffers of their own.  Such a launch is bound by a weight wave's chain, ~220 instructions per K step at one wave on its SIMD
// (which issues one every ~6 cycles); with two waves per SIMD half as many steps stand one behind the other.  Either half keeps
// the sums of half of the tile's rows.
//
// BLK: the matrix instruction, 16x16x32 or 32x32x16 (see below).  GROUPED: a grouped launch, which never writes y.
template <int WAVES_M, int WAVES_N, int WMB, int WNB, int DT, bool FUSE_LOSS, int FMT, bool DUAL = false, int KS = 1, int BLK = 16, bool GROUPED = false, int SHARED = kNotShared>
__device__ __forceinline__ void linear_fwd_body(const FwdParams& p, const int bm, const int bn,
                                                const uint32_t __attribute__((address_space(4)))* entry = nullptr) {
  constexpr int NWAVES = WAVES_M * WAVES_N;
  constexpr int BM = 32 * WMB * WAVES_M, BN = 32 * WNB * WAVES_N;
  constexpr int TN = DUAL ? BN / 2 : BN;           // output columns of the tile
  static_assert(!DUAL || (FUSE_LOSS && FMT == SZO_FORMAT_UNIFORM && BN == 256), "dual-sign tiles: fused loss, uniform format, 256 rows");
  constexpr int W_WAVES = BN / 64;                 // one per 64-row band of the weight tile
  constexpr int X_WAVES = NWAVES - W_WAVES;
  static_assert(BN % 64 == 0 && X_WAVES > 0, "need whole bands and at least one activation wave");
  constexpr int X_ROWS_PER_PASS = 8 * X_WAVES;     // 8 lanes cover one 128-byte row of x
  static_assert(BM == 8 * X_ROWS_PER_PASS, "every activation lane stages 8 chunks per tile");
  constexpr int SLOTS = 4 * WMB * WNB;             // pairs of 16x16x32 MFMAs per K step
  constexpr int SPU = SLOTS / 8;                   // slots per activation staging unit: 1, 2 or 4
  constexpr int WPS = 4 / SPU;                     // output words produced per slot
  // Weight waves finish their dense staging in the first three quarters of the slots (32 slots: 3 per unit; 16 slots: 3 per
  // two units) and spend the rest on the sensitive entries of the tile, so that the dependent LDS
  // round trips of the scatter also run in the shadow of MFMAs instead of after them (16 slots: forwards of a Llama block's linears
  // at 600 tokens 513 -> 486 us, a 3000 x 4096 layer at 560 tokens and 1 % 68 -> 63, a 4096 x 4096 composed step at 1000 128 -> 121).
  static_assert(SLOTS == 32 || SLOTS == 16, "two schedules exist");
  constexpr int SC_WINDOW = SLOTS == 32 ? 24 : 6, SC_READ = SLOTS == 32 ? 27 : 12, SC_STORE = SLOTS == 32 ? 30 : 15;
  typedef typename Frag<DT>::type frag_t;

  static_assert(KS == 1 || (KS == 2 && SLOTS == 16 && !DUAL && FMT == SZO_FORMAT_UNIFORM), "K in two parts: the small tile");
  extern __shared__ __attribute__((aligned(16))) uint16_t smem[];
  const int tid = threadIdx.x, lane = tid & 63;
  const int any_wave = __builtin_amdgcn_readfirstlane(tid >> 6), kpart = KS == 1 ? 0 : any_wave / NWAVES;
  // (the second part's weight waves share their SIMDs with the first part's activation waves)
  const int wave = KS == 1 ? any_wave : (any_wave % NWAVES) ^ (kpart ? NWAVES / 2 : 0);
  uint16_t* const lds = smem + kpart * (tiled_lds_bytes(BM, BN) / 2);
  uint16_t* const ldsA = lds;                                   // [2][BM*BK]
  uint16_t* const ldsB = lds + 2 * BM * BK;                     // [2][BN*BK]
  float* const winVal = reinterpret_cast<float*>(lds + 2 * (BM + BN) * BK);        // [W_WAVES][kWindow]
  uint16_t* const winPos = reinterpret_cast<uint16_t*>(winVal + W_WAVES * kWindow);  // [W_WAVES][kWindow]
  uint16_t* const sink16 = winPos + W_WAVES * kWindow;                              // [W_WAVES][64] write sink of idle lanes

  const int wm = wave / WAVES_N, wn = wave % WAVES_N;
  const int m0 = bm * BM, n0 = bn * TN;
  const int nk = p.ktiles / KS, k0 = kpart * nk;            // this part's K steps: k0 .. k0 + nk - 1 (whole parts, checked on the host)
  // Fields that are only needed now and then (a window refill every ~64 K steps, the loss epilogue) are read
  // again from the table entry where they are used instead of occupying scalar registers for the whole
  // tile; the pointer is laundered so that the loads stay where they are written.  Only with dual-sign
  // tiles: otherwise the grouped launch has changed `p` for the -eps forward.
  auto cold = [&]() -> FwdParams {
    if (!(DUAL || SHARED) || entry == nullptr) return p;
    constexpr int W = (int)(sizeof(FwdParams) / 4);
    const uint32_t __attribute__((address_space(4)))* e = entry;
    asm volatile("" : "+s"(e));
    struct Words { uint32_t w[W]; } raw;
#pragma unroll
    for (int i = 0; i < W; ++i) raw.w[i] = e[i];
    return __builtin_bit_cast(FwdParams, raw);
  };

  // Blocks of 16 x 16 outputs.  At the sizes that fill the chip this kernel runs at the chip's power limit, and 16x16x32 takes
  // less power per product than 32x32x16 (half the accumulator traffic): a bare loop with the kernel's operands, operand reads
  // and four vector instructions per 32 768 FLOP reaches 1566 against 1411 TFLOP/s, and the step over four Llama blocks
  // runs at 1.86 GHz instead of 1.69 for 5 % more cycles.  us, 32x32x16 -> 16x16x32: two Llama blocks at 4096 tokens 5358 -> 5120, with
  // the bf16 tile 5528 -> 5212, with tables 5880 -> 5685; one Mistral block at 8192 and 1 % 6148 -> 5836; two of them with two sets of
  // activations at 333 701 -> 661; a 4096 x 4096 composed step at 2000 176 -> 167.
  // Blocks of 32 x 32: half as many instructions, for launches that are bound by a weight wave's instructions and not by power
  // (see wide_blocks, kFewTableTiles).
  // RING operands of x are held at a time, each re-read for a later row of blocks as soon as its own has been issued: three are
  // what the registers of the 32-slot schedule allow with 16 x 16, four hide more where one wave has a SIMD to itself (six forwards of a Llama
  // block at 600 tokens 501 -> 494; 32 x 32 with tables in half-empty tiles, 5087 x 6208 at 14 tokens 104.3 -> 103.6).
  static_assert(BLK == 16 || (BLK == 32 && KS == 1 && !DUAL && (SLOTS == 16 || FMT == SZO_FORMAT_LUT)), "32 x 32: whole small tiles and tables");
  constexpr int NA = 32 * WMB / BLK, NB = 32 * WNB / BLK, KSTEPS = BLK / 8, LANE_SHIFT = BLK == 16 ? 4 : 5, RING = SLOTS == 32 && BLK == 16 ? 3 : 4;
  typedef typename std::conditional<BLK == 16, float4_t, float16_t>::type acc_t;
  acc_t acc[NA][NB];
#pragma unroll
  for (int i = 0; i < NA; ++i)
#pragma unroll
    for (int j = 0; j < NB; ++j)
#pragma unroll
      for (int r = 0; r < BLK * BLK / 64; ++r) acc[i][j][r] = 0.0f;

  // Lane l of an operand holds row l % BLK of its block, columns 8 (l / BLK) .. of a step: a chunk of the staged row.
  const int fragA_row = wm * 32 * WMB + (lane & (BLK - 1)), fragB_row = wn * 32 * WNB + (lane & (BLK - 1));
  auto read_a = [&](int buf, int ks, int i) -> frag_t {
    return *reinterpret_cast<const frag_t*>(ldsA + buf * BM * BK + chunk_off(fragA_row, 64 / BLK * ks + (lane >> LANE_SHIFT)) + BLK * i * BK);
  };
  auto read_b = [&](int buf, int ks, int j) -> frag_t {
    return *reinterpret_cast<const frag_t*>(ldsB + buf * BN * BK + chunk_off(fragB_row, 64 / BLK * ks + (lane >> LANE_SHIFT)) + BLK * j * BK);
  };

  // All MFMAs of one K step on buffer buf, with slice(s) issued behind every second one (32 x 32: behind each).
  auto run_tile = [&](int buf, auto&& slice) {
    constexpr int PER_SLOT = BLK == 16 ? 2 : 1;
    frag_t a[RING], b[2][NB];
    a[0] = read_a(buf, 0, 0);
#pragma unroll
    for (int j = 0; j < NB; ++j) b[0][j] = read_b(buf, 0, j);
#pragma unroll
    for (int i = 1; i < RING; ++i) a[i] = read_a(buf, i / NA, i % NA);
#pragma unroll
    for (int ks = 0; ks < KSTEPS; ++ks) {
#pragma unroll
      for (int i = 0; i < NA; ++i) {
#pragma unroll
        for (int j = 0; j < NB; ++j) {
          const int at = ks * NA + i, m = at * NB + j;
          if constexpr (BLK == 16) acc[i][j] = Frag<DT>::mfma16(a[at % RING], b[ks & 1][j], acc[i][j]);
          else acc[i][j] = Frag<DT>::mfma(a[at % RING], b[ks & 1][j], acc[i][j]);
          if (ks + 1 < KSTEPS && i == (BLK == 16 ? NA / 2 : 0)) b[(ks + 1) & 1][j] = read_b(buf, ks + 1, j);
          if (j == NB - 1 && at + RING < KSTEPS * NA) a[at % RING] = read_a(buf, (at + RING) / NA, (at + RING) % NA);
          if (m % PER_SLOT == PER_SLOT - 1) {
            slice(m / PER_SLOT);
            __builtin_amdgcn_sched_barrier(0);
          }
        }
      }
    }
  };

  if (DUAL && wave >= W_WAVES / 2 && wave < W_WAVES) {
    // ============ DUAL: the bands of these waves are the -eps copies, written by waves 0 .. W_WAVES/2-1 ====
    auto nothing = [](int) {};
    for (int kt = 0; kt < nk; kt += 2) {
      __syncthreads();
      run_tile(0, nothing);
      if (kt + 1 < nk) {
        __syncthreads();
        run_tile(1, nothing);
      }
    }
  } else if (wave < W_WAVES) {
    // =============================== weight wave ===============================================
    // Lane l stages row l of the band: all 64 columns of a tile, as two halves i = 0, 1 of 32 columns
    // (16 bytes of codes, one scale each).  A wave-wide write of one chunk then touches 64 consecutive rows
    // at the same logical chunk -- the access pattern of the operand reads, which the swizzle makes
    // conflict-free (with two lanes per row the writes measured two-way bank conflicts).
    const int wr = wave * 64 + lane;                             // tile row
    const int band = n0 / 64 + wave;                             // band of the sparse layout
    const bool band_ok = band < p.bands;
    const uint32_t tp_base = (uint32_t)band * (uint32_t)p.ktiles + (uint32_t)k0;
    uint32_t tile_lo = 0, band_end = 0;                          // entry range bookkeeping (uniform)
    uint32_t tp_reg = 0;                                         // lane l: tile_ptr[tp_base + 64*c + 1 + l]
    uint32_t t_lo = 0, t_end = 0;
    if (band_ok) {
      // Three independent loads and (below, after the first codes have been requested too) one wait: the
      // tile's first K step cannot start before the band's first entries are known, so every memory
      // round trip here is dead time for the whole workgroup.
      t_lo = p.tile_ptr[tp_base];
      t_end = p.tile_ptr[tp_base + nk];
      tp_reg = p.tile_ptr[min(tp_base + 1u + (uint32_t)lane, tp_base + (uint32_t)nk)];
    }
    uint32_t win_lo = 0, win_hi = 0;                             // entries [win_lo, win_hi) are in the window
    float* const wv = winVal + wave * kWindow;
    float* const wv_minus = winVal + (wave + W_WAVES / 2) * kWindow;   // DUAL: value for the -eps copy (the idle waves' space)
    uint16_t* const wp = winPos + wave * kWindow;
    constexpr int kMinusCopy = (BN / 2) * BK;                    // DUAL: offset of the -eps copy of a tile position (128 rows:
                                                                 // the swizzle, a function of row mod 16, is the same there)

    // Banded layout: the 64 rows of this wave's band, one 64-column tile, are 2 KB in a row, so the two
    // load instructions of the wave (64 rows x 16 bytes each) cover it without gaps.  Bands past N re-read the
    // last band (their outputs are never stored) and column tiles past the end re-read the last
    // tile (never consumed): the loads stay unconditional and in order.
    global_u8 qrow[2];
    global_u16 srow[2];
    {
      const size_t bsafe = (size_t)min(band, p.bands - 1);
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        const int r = lane;                                        // row inside the band
        qrow[i] = p.qweight + ((bsafe * (size_t)p.ktiles + (size_t)k0) * 64 + (size_t)r) * 32 + 16 * i;
        srow[i] = p.scales + bsafe * (size_t)(p.K >> p.group_shift) * 64 + (size_t)((r & 15) * 4 + (r >> 4));
      }
    }
    u32x4 qreg[2];
    uint16_t sreg[2];
    DequantConsts dqk;
    dqk.magic_lo = 0x64006400u; dqk.magic_hi = 0x54005400u;
    asm volatile("" : "+v"(dqk.magic_lo), "+v"(dqk.magic_hi));   // keep them in registers, not as literals
    auto load_q = [&](int kt, int i) {
      qreg[i] = *reinterpret_cast<global_u32x4>(qrow[i] + (size_t)min(kt, nk - 1) * (64 * BK / 2));
    };
    auto load_s = [&](int kt, int i) {
      sreg[i] = srow[i][(size_t)(((k0 + min(kt, nk - 1)) * BK + 32 * i) >> p.group_shift) * 64];
    };
    auto load_w = [&](int kt, int i) { load_q(kt, i); load_s(kt, i); };

    // Slice s of staging the registers into buffer dst while reloading them with tile load_kt.
    // Unit u = s / SPU is code word u%4 of row half u/4; each slot produces WPS of its 4 words.
    // ---- sensitive entries -------------------------------------------------------------------
    // Computes entries [s, s+256) of the band (s a multiple of 4) into the window.
    auto refill = [&](uint32_t s) {
      const FwdParams pr = cold();
      const uint32_t j = s + 4u * lane;
      if (j < band_end) {
        uint32_t idx[4];
        float val[4];
        if (j + 3 < pr.nnz) {
          const u32x4 iv = *reinterpret_cast<global_u32x4>(pr.sp_idx + j);
          const u32x4 vv = *reinterpret_cast<global_u32x4>(pr.sp_val + j);
#pragma unroll
          for (int c = 0; c < 4; ++c) { idx[c] = iv[c]; val[c] = __uint_as_float(vv[c]); }
        } else {
#pragma unroll
          for (int c = 0; c < 4; ++c) {
            const bool ok = j + c < pr.nnz;
            idx[c] = ok ? pr.sp_idx[j + c] : 0xFFFFFFFFu;
            val[c] = ok ? pr.sp_val[j + c] : 0.0f;
          }
        }
        float val_minus[4] = {val[0], val[1], val[2], val[3]};
        if (!SHARED && pr.signed_eps != 0.0f) {
          float z[4];
          zbar_quad((pr.nnz_base + j) >> 2, pr.seed, pr.step, z);
#pragma unroll
          for (int c = 0; c < 4; ++c) {
            if (DUAL) val_minus[c] = fmaf(-pr.signed_eps, z[c], val[c]);
            val[c] = fmaf(pr.signed_eps, z[c], val[c]);
          }
        }
#pragma unroll
        for (int c = 0; c < 4; ++c) {
          const uint32_t n = fast_div(idx[c], pr.div_mul, pr.div_shift);
          const uint32_t r = n - (uint32_t)(band * 64);                   // row inside the band
          const uint32_t kk = (idx[c] - n * (uint32_t)pr.K) & 63u;
          wp[4 * lane + c] = (r < 64u) ? (uint16_t)lds_pos<DT>(wave * 64 + (int)r, (int)kk) : (uint16_t)0xFFFFu;
          wv[4 * lane + c] = val[c];
          if (DUAL) wv_minus[4 * lane + c] = val_minus[c];
        }
      }
      win_lo = s;
      win_hi = min(s + (uint32_t)kWindow, band_end);
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");     // window visible to the other lanes of the wave
    };

    // General path: adds entries [lo, hi) of the band into LDS buffer `buf`, any count.
    auto scatter_range = [&](uint32_t lo, uint32_t hi_end, int buf) {
      uint16_t* B = ldsB + buf * BN * BK;
      uint32_t cur = lo;
      while (cur < hi_end) {
        if (cur >= win_hi || cur < win_lo) refill(cur & ~3u);
        const uint32_t hi = min(hi_end, win_hi);
        for (uint32_t j = cur + lane; j < hi; j += 64) {
          const uint32_t e = j - win_lo;
          const uint32_t pos = wp[e];
          if (pos != 0xFFFFu) {
            uint16_t* w = B + pos;
            Frag<DT>::store(w, Frag<DT>::load(w) + wv[e]);
            if (DUAL) Frag<DT>::store(w + kMinusCopy, Frag<DT>::load(w + kMinusCopy) + wv_minus[e]);
          }
        }
        cur = hi;
      }
    };

    // Per-tile bookkeeping, done before the MFMA loop that stages the tile.  Tiles with at most 64
    // entries (the normal case) take the in-slot path: sc_cnt entries starting at window offset
    // sc_e0, one per lane.  Of larger tiles the 16-slot schedule takes the first 64 that way and leaves the rest to
    // scatter_range after the loop; the 32-slot one leaves all of them to it.  A forward with 1 % of sensitive weights, half of them in
    // 1 % of the rows, us with the whole tile / the rest of it behind the loop: 4096 x 4096 at 450 tokens 89 / 81, 1024 x 4096 at
    // 700 80 / 71, 4096 x 11008 at 1200 261 / 249 (32 slots: a Llama block's step at 4096 tokens takes 0.7 % longer with the rest behind it).
    uint32_t sc_cnt = 0, sc_e0 = 0, big_lo = 0, big_hi = 0;
    auto prepare_scatter = [&](int kt) {
      sc_cnt = 0; big_lo = 0; big_hi = 0;
      if (!band_ok || kt >= nk) return;
      if ((kt & 63) == 0 && kt > 0) {                        // the first 64 boundaries were loaded with tile_lo
        const uint32_t t = tp_base + (uint32_t)kt + 1u + lane;
        tp_reg = (t <= tp_base + (uint32_t)nk) ? cold().tile_ptr[t] : band_end;
        asm volatile("" : "+v"(tp_reg));       // consume the load here, so that no wait on it is needed later
      }
      const uint32_t hi = __builtin_amdgcn_readlane(tp_reg, kt & 63), lo = tile_lo;
      tile_lo = hi;
      if (hi <= lo) return;
      if (SLOTS == 16) {
        const uint32_t first = min(hi, lo + 64u);
        if (lo < win_lo || first > win_hi) refill(lo & ~3u);
        sc_cnt = first - lo;
        sc_e0 = lo - win_lo;
        big_lo = first; big_hi = hi;
      } else if (hi - lo <= 64u) {
        if (lo < win_lo || hi > win_hi) refill(lo & ~3u);
        sc_cnt = hi - lo;
        sc_e0 = lo - win_lo;
      } else {
        big_lo = lo; big_hi = hi;
      }
    };

    if constexpr (FMT == SZO_FORMAT_LUT) {
      // ---- table format: dq[n,k] = lut[n][code] (non-uniform 4-bit quantisers, Appendix C.5) -------
      // gfx950 has no register-indexed look-up, so the table of a row is held as four byte planes (low
      // and high bytes of entries 0-7 and of entries 8-15, two registers each) and looked up with the
      // byte-permute instruction, four codes at a time: low 3 bits of the codes select inside a plane,
      // bit 3 picks the plane.  That only pays if a lane keeps ONE row's table for the whole K loop:
      // lane l stages row l of the band, all 64 columns of a tile (32 bytes of codes, two 16-byte loads).
      static_assert(DT == SZO_TILE_F16 && SLOTS == 32, "table format: fp16 tile, 32-slot schedule");
      const int lrow = wave * 64 + lane;                           // row of the weight tile
      const global_u8 qr = p.qweight + ((size_t)min(band, p.bands - 1) * (size_t)nk * 64 + (size_t)lane) * 32;
      u32x4 qv[2];
      auto load_qv = [&](int kt, int h) {
        qv[h] = *reinterpret_cast<global_u32x4>(qr + (size_t)min(kt, nk - 1) * (64 * BK / 2) + 16 * h);
      };
      uint32_t lo_a0, lo_a1, lo_b0, lo_b1, hi_a0, hi_a1, hi_b0, hi_b1;
      {
        // rows past N re-read the last row's table: their outputs are never used
        const global_u32x4 lp = reinterpret_cast<global_u32x4>(p.lut + (size_t)min(n0 + lrow, p.N - 1) * 16);
        const u32x4 a = lp[0], b = lp[1];                          // entries 0-7 and 8-15, two per word
        lo_a0 = __builtin_amdgcn_perm(a[1], a[0], 0x06040200u); lo_a1 = __builtin_amdgcn_perm(a[3], a[2], 0x06040200u);
        hi_a0 = __builtin_amdgcn_perm(a[1], a[0], 0x07050301u); hi_a1 = __builtin_amdgcn_perm(a[3], a[2], 0x07050301u);
        lo_b0 = __builtin_amdgcn_perm(b[1], b[0], 0x06040200u); lo_b1 = __builtin_amdgcn_perm(b[3], b[2], 0x06040200u);
        hi_b0 = __builtin_amdgcn_perm(b[1], b[0], 0x07050301u); hi_b1 = __builtin_amdgcn_perm(b[3], b[2], 0x07050301u);
      }
      // Slots 3d, 3d+1, 3d+2 turn code word d (columns 8d .. 8d+7) into chunk d of the row:
      //   selectors and plane masks  ->  eight look-ups and four selects  ->  interleave and store.
      // Even codes (0,2,4,6) sit in the low nibbles of the word's bytes, odd ones in the high nibbles;
      // the chunk keeps the element order (0,4)(1,5)(2,6)(3,7) that the activations are staged in.
      // Slots 24, 27 and 30 scatter the tile's sensitive entries as in the uniform format.
      uint32_t sel_e = 0, sel_o = 0, m_e = 0, m_o = 0, lo_e = 0, hi_e = 0, lo_o = 0, hi_o = 0;
      u32x4 outw;
      uint32_t sc_pos = 0xFFFFu;
      float sc_val = 0.0f, sc_old = 0.0f;
      uint16_t* sc_addr = nullptr;
      auto make_slice = [&](int dst, int load_kt) {
        return [&, dst, load_kt](int s) {
          if (s < 24) {
            const int d = s / 3, ph = s % 3;
            if (ph == 0) {
              const uint32_t q = qv[d >> 2][d & 3];
              sel_e = q & 0x07070707u;
              sel_o = (q >> 4) & 0x07070707u;
              // 0xFF in the bytes whose code has bit 3 set: byte 1 of the constant, else byte 0
              m_e = __builtin_amdgcn_perm(0u, 0x0000FF00u, (q >> 3) & 0x01010101u);
              m_o = __builtin_amdgcn_perm(0u, 0x0000FF00u, (q >> 7) & 0x01010101u);
              if ((d & 3) == 3) load_qv(load_kt, d >> 2);          // codes consumed: reload in place
            } else if (ph == 1) {
              auto pick = [](uint32_t m, uint32_t b, uint32_t a) { return (m & b) | (~m & a); };
              lo_e = pick(m_e, __builtin_amdgcn_perm(lo_b1, lo_b0, sel_e), __builtin_amdgcn_perm(lo_a1, lo_a0, sel_e));
              hi_e = pick(m_e, __builtin_amdgcn_perm(hi_b1, hi_b0, sel_e), __builtin_amdgcn_perm(hi_a1, hi_a0, sel_e));
              lo_o = pick(m_o, __builtin_amdgcn_perm(lo_b1, lo_b0, sel_o), __builtin_amdgcn_perm(lo_a1, lo_a0, sel_o));
              hi_o = pick(m_o, __builtin_amdgcn_perm(hi_b1, hi_b0, sel_o), __builtin_amdgcn_perm(hi_a1, hi_a0, sel_o));
            } else {
              outw[0] = __builtin_amdgcn_perm(hi_e, lo_e, 0x06020400u);      // codes 0, 4
              outw[1] = __builtin_amdgcn_perm(hi_o, lo_o, 0x06020400u);      // codes 1, 5
              outw[2] = __builtin_amdgcn_perm(hi_e, lo_e, 0x07030501u);      // codes 2, 6
              outw[3] = __builtin_amdgcn_perm(hi_o, lo_o, 0x07030501u);      // codes 3, 7
              *reinterpret_cast<u32x4*>(ldsB + dst * BN * BK + chunk_off(lrow, d)) = outw;
            }
          }
          const bool active = (uint32_t)lane < sc_cnt;
          if (s == 24) {
            const uint32_t e = active ? sc_e0 + lane : 0u;
            sc_pos = wp[e];
            sc_val = wv[e];
          } else if (s == 27) {                         // every dense word of the tile is written by slot 23
            const bool ok = active && sc_pos != 0xFFFFu;
            sc_addr = ok ? ldsB + dst * BN * BK + sc_pos : sink16 + wave * 64 + lane;
            sc_val = ok ? sc_val : 0.0f;
            sc_old = Frag<DT>::load(sc_addr);
          } else if (s == 30) {
            Frag<DT>::store(sc_addr, sc_old + sc_val);
          }
        };
      };

      __builtin_amdgcn_s_setprio(1);
      load_qv(0, 0);
      load_qv(0, 1);
      tile_lo = __builtin_amdgcn_readfirstlane(t_lo);
      band_end = __builtin_amdgcn_readfirstlane(t_end);
      prepare_scatter(0);
      {
        auto slice = make_slice(0, 1);
#pragma unroll
        for (int s = 0; s < SLOTS; ++s) slice(s);
      }
      if (big_hi > big_lo) scatter_range(big_lo, big_hi, 0);
      for (int kt = 0; kt < nk; kt += 2) {
        __syncthreads();                       // tile kt complete in buffer 0; buffer 1 no longer read
        prepare_scatter(kt + 1);
        run_tile(0, make_slice(1, kt + 2));
        if (big_hi > big_lo) scatter_range(big_lo, big_hi, 1);
        if (kt + 1 < nk) {
          __syncthreads();
          prepare_scatter(kt + 2);
          run_tile(1, make_slice(0, kt + 3));
          if (big_hi > big_lo) scatter_range(big_lo, big_hi, 0);
        }
      }
    } else {
    // ---- slices ---------------------------------------------------------------------------------
    // Dense part: unit u = code word u%4 of row half u/4; the unit's four output words are spread 2,1,1 over three slots, with
    // 16 slots the eight words of two units 3,3,2.  In the 32-slot schedule the
    // three instructions of an output word (and_or, subtract offset, multiply by scale) run in
    // three consecutive slots, so no slot holds two dependent VALU instructions.
    // Scatter part: window read, tile read (behind the last dense write), add + write, three slots
    // or more apart; lanes without an entry go through a per-lane sink in LDS, which keeps it branch-free.
    constexpr int PIPE = SLOTS == 32 ? 1 : 0;      // slot distance between the stages of a word
    u32x4 outw;
    uint32_t st_a[3][2], st_b[3][2];
    uint32_t sc_pos = 0xFFFFu;
    float sc_val = 0.0f, sc_old = 0.0f, sc_val_minus = 0.0f, sc_old_minus = 0.0f;
    uint16_t* sc_addr = nullptr;
    uint16_t* sc_addr_minus = nullptr;
    auto make_slice = [&](int dst, int load_kt) {
      return [&, dst, load_kt](int s) {
        // the k-th output word (of two, three with 16 slots) staged from slot `slot`: unit u, word w; false if none
        auto item = [](int slot, int k, int& u, int& w) -> bool {
          if (slot < 0 || slot >= SLOTS / 4 * 3) return false;
          const int ph = slot % 3;
          const int w0 = SLOTS == 32 ? (ph == 0 ? 0 : ph + 1) : 3 * ph;
          const int nw = SLOTS == 32 ? (ph == 0 ? 2 : 1) : (ph < 2 ? 3 : 2);
          u = SLOTS == 32 ? slot / 3 : 2 * (slot / 3) + ((w0 + k) >> 2);
          w = (w0 + k) & 3;
          return k < nw;
        };
        constexpr int KMAX = SLOTS == 32 ? 2 : 3;
        static_assert(KMAX <= 2 || PIPE == 0, "stage registers hold two words per slot");
        // All three stages in one slot, its words side by side: word by word the compiler puts an empty instruction between dependent
        // packed-half ones, 16 of the 227 of a K step (six forwards of a Llama block at 600 tokens 518 -> 507 us).
        if (PIPE == 0) {
          uint32_t word[KMAX];
          if (DT == SZO_TILE_F16) {
#pragma unroll
            for (int k = 0; k < KMAX; ++k) {
              int u = 0, w = 0;
              if (!item(s, k, u, w)) continue;
              const uint32_t q = qreg[u >> 2][u & 3];
              word[k] = and_or(w < 2 ? q : (q >> 8), (w & 1) ? 0x00F000F0u : 0x000F000Fu, (w & 1) ? dqk.magic_hi : dqk.magic_lo);
            }
#pragma unroll
            for (int k = 0; k < KMAX; ++k) {
              int u = 0, w = 0;
              if (!item(s, k, u, w)) continue;
              const _Float16 o = (w & 1) ? (_Float16)72.0f : (_Float16)1032.0f;
              word[k] = __builtin_bit_cast(uint32_t, __builtin_bit_cast(half2_t, word[k]) - half2_t{o, o});
            }
          }
#pragma unroll
          for (int k = 0; k < KMAX; ++k) {
            int u = 0, w = 0;
            if (!item(s, k, u, w)) continue;
            const int i = u >> 2, c = u & 3;
            const _Float16 sh = __builtin_bit_cast(_Float16, sreg[i]);
            if (DT == SZO_TILE_F16) outw[w] = __builtin_bit_cast(uint32_t, __builtin_bit_cast(half2_t, word[k]) * half2_t{sh, sh});
            else outw[w] = dequant_out<DT>(qreg[i][c], w, (float)sh, half2_t{sh, sh}, dqk);
            if (w == 3) {
              *reinterpret_cast<u32x4*>(ldsB + dst * BN * BK + chunk_off(wr, 4 * i + c)) = outw;
              if (DUAL) *reinterpret_cast<u32x4*>(ldsB + dst * BN * BK + kMinusCopy + chunk_off(wr, 4 * i + c)) = outw;
              if (c == 3) load_w(load_kt, i);
            }
          }
        }
#pragma unroll
        for (int k = 0; PIPE != 0 && k < KMAX; ++k) {
          int u = 0, w = 0;
          if (item(s, k, u, w)) {                       // stage A: isolate the nibble pair under its exponent
            const int i = u >> 2, c = u & 3;
            const uint32_t q = qreg[i][c];
            if (DT == SZO_TILE_F16)
              st_a[s % 3][k] = and_or(w < 2 ? q : (q >> 8), (w & 1) ? 0x00F000F0u : 0x000F000Fu,
                                      (w & 1) ? dqk.magic_hi : dqk.magic_lo);
            if (w == 3 && c == 3 && DT == SZO_TILE_F16) load_q(load_kt, i);   // codes consumed: reload in place
          }
          if (item(s - 1, k, u, w) && DT == SZO_TILE_F16) {   // stage B: remove the exponent's offset (exact)
            const _Float16 o = (w & 1) ? (_Float16)72.0f : (_Float16)1032.0f;
            const half2_t h = __builtin_bit_cast(half2_t, st_a[(s - 1) % 3][k]) - half2_t{o, o};
            st_b[(s - 1) % 3][k] = __builtin_bit_cast(uint32_t, h);
          }
          if (item(s - 2, k, u, w)) {                   // stage C: scale, rounded once
            const int i = u >> 2, c = u & 3;
            const _Float16 sh = __builtin_bit_cast(_Float16, sreg[i]);
            if (DT == SZO_TILE_F16) {
              const half2_t h = __builtin_bit_cast(half2_t, st_b[(s - 2) % 3][k]) * half2_t{sh, sh};
              outw[w] = __builtin_bit_cast(uint32_t, h);
            } else {
              outw[w] = dequant_out<DT>(qreg[i][c], w, (float)sh, half2_t{sh, sh}, dqk);
            }
            if (w == 3) {
              *reinterpret_cast<u32x4*>(ldsB + dst * BN * BK + chunk_off(wr, 4 * i + c)) = outw;
              if (DUAL) *reinterpret_cast<u32x4*>(ldsB + dst * BN * BK + kMinusCopy + chunk_off(wr, 4 * i + c)) = outw;
              if (c == 3) {
                if (DT != SZO_TILE_F16) load_q(load_kt, i);
                load_s(load_kt, i);
              }
            }
          }
        }
        {
          const bool active = (uint32_t)lane < sc_cnt;
          if (s == SC_WINDOW) {
            const uint32_t e = active ? sc_e0 + lane : 0u;
            sc_pos = wp[e];
            sc_val = wv[e];
            if (DUAL) sc_val_minus = wv_minus[e];
          } else if (s == SC_READ) {                         // every dense word of the tile has been written
            const bool ok = active && sc_pos != 0xFFFFu;
            sc_addr = ok ? ldsB + dst * BN * BK + sc_pos : sink16 + wave * 64 + lane;
            sc_val = ok ? sc_val : 0.0f;
            sc_old = Frag<DT>::load(sc_addr);
            if (DUAL) {                                 // the same position in the -eps copy
              sc_addr_minus = ok ? ldsB + dst * BN * BK + kMinusCopy + sc_pos : sink16 + (wave + W_WAVES / 2) * 64 + lane;
              sc_val_minus = ok ? sc_val_minus : 0.0f;
              sc_old_minus = Frag<DT>::load(sc_addr_minus);
            }
          } else if (s == SC_STORE) {
            Frag<DT>::store(sc_addr, sc_old + sc_val);
            if (DUAL) Frag<DT>::store(sc_addr_minus, sc_old_minus + sc_val_minus);
          }
        }
      };
    };

    // Weight waves carry more staging instructions per MFMA slot than activation waves; a higher
    // issue priority lets the two waves of a SIMD finish their K step together.
    __builtin_amdgcn_s_setprio(1);
    load_w(0, 0);
    load_w(0, 1);
    tile_lo = __builtin_amdgcn_readfirstlane(t_lo);
    band_end = __builtin_amdgcn_readfirstlane(t_end);
    prepare_scatter(0);
    {
      auto slice = make_slice(0, 1);
#pragma unroll
      for (int s = 0; s < SLOTS; ++s) slice(s);
    }
    if (big_hi > big_lo) scatter_range(big_lo, big_hi, 0);
    for (int kt = 0; kt < nk; kt += 2) {
      __syncthreads();                       // tile kt complete in buffer 0; buffer 1 no longer read
      prepare_scatter(kt + 1);
      run_tile(0, make_slice(1, kt + 2));
      if (big_hi > big_lo) scatter_range(big_lo, big_hi, 1);
      if (kt + 1 < nk) {
        __syncthreads();
        prepare_scatter(kt + 2);
        run_tile(1, make_slice(0, kt + 3));
        if (big_hi > big_lo) scatter_range(big_lo, big_hi, 0);
      }
    }
    }  // uniform format
  } else {
    // =============================== activation wave ===========================================
    const int xt = 64 * wave + lane - 64 * W_WAVES;
    const int xc = xt & 7, xr = xt >> 3;                       // chunk, row (plus X_ROWS_PER_PASS*u)
    u32x4 xreg[8];
    // SHARED: a buffer of the tile's rows and one offset instead of eight pointers, whose registers its epilogue has no room for.  Rows past M
    // are out of its bounds and read as zero; what is loaded past the end of a row is not used.
    global_u16 xrow[8];
#pragma unroll
    for (int u = 0; u < 8; ++u)
      xrow[u] = p.x + (size_t)min(m0 + xr + X_ROWS_PER_PASS * u, p.M - 1) * p.K + k0 * BK + xc * 8;
    const __amdgpu_buffer_rsrc_t xbuf = __builtin_amdgcn_make_buffer_rsrc((void*)(uintptr_t)(p.x + (size_t)m0 * p.K), 0, min(p.M - m0, BM) * 2 * p.K, 0x00027000);
    const int xoff = xr * 2 * p.K + 16 * xc;
    auto load_x = [&](int kt, int u) {
      if (SHARED) xreg[u] = __builtin_amdgcn_raw_buffer_load_b128(xbuf, xoff + (X_ROWS_PER_PASS * u * 2 * p.K + kt * (2 * BK)), 0, 0);
      else xreg[u] = *reinterpret_cast<global_u32x4>(xrow[u] + min(kt, nk - 1) * BK);
    };
    u32x4 outw;
    auto make_slice = [&](int dst, int load_kt) {
      return [&, dst, load_kt](int s) {
        const int u = s / SPU;
#pragma unroll
        for (int o = 0; o < WPS; ++o) {
          const int w = (s % SPU) * WPS + o;
          outw[w] = stage_x_word<DT>(xreg[u], w);
        }
        if (s % SPU == SPU - 1) {
          *reinterpret_cast<u32x4*>(ldsA + dst * BM * BK + chunk_off(xr + X_ROWS_PER_PASS * u, xc)) = outw;
          load_x(load_kt, u);
        }
      };
    };

#pragma unroll
    for (int u = 0; u < 8; ++u) load_x(0, u);
    {
      auto slice = make_slice(0, 1);
#pragma unroll
      for (int s = 0; s < SLOTS; ++s) slice(s);
    }
    static_assert(WAVES_M == 2 && X_WAVES == WAVES_N, "the activation waves are those of the lower half of the tile");
    if (!DUAL && p.M - m0 <= BM / 2) {
      // Last row of tiles, half or more of it padding: these waves' outputs are all padding.  They stage the rows of the upper half
      // and leave the matrix cores to the weight waves, which halves what bounds a K step.  Two Mistral blocks with two sets of
      // activations at 333 tokens (77 rows in the second row of tiles) 797 -> 672 us per step, six forwards of an OPT block at 777
      // 544 -> 535; with the table format, whose K step is bound by the look-ups, no change.  Not with dual-sign tiles: launches of
      // many rows, and registers spilled in the schedule below (8 instead of 6).
#pragma unroll 1
      for (int kt = 0; kt < nk; ++kt) {
        __syncthreads();
        int dst = (kt + 1) & 1;
        asm volatile("" : "+s"(dst));                       // addresses are formed here, not held through the other branch
        auto slice = make_slice(dst, kt + 2);
#pragma unroll
        for (int s = 0; s < SLOTS / 2; ++s) slice(s);
      }
    } else {
      for (int kt = 0; kt < nk; kt += 2) {
        __syncthreads();
        run_tile(0, make_slice(1, kt + 2));
        if (kt + 1 < nk) {
          __syncthreads();
          run_tile(1, make_slice(0, kt + 3));
        }
      }
    }
  }

  if constexpr (SHARED) {
    static_assert(!DUAL && KS == 1 && BLK == 16 && BM == 256 && BN == 256 && FUSE_LOSS, "256 x 256 outputs, one launch for both signs");
    shared_tail<DT, SHARED == kSharedFp64Sums>(acc, cold, bm, bn, reinterpret_cast<uint8_t*>(smem));
    return;
  }
  // ---- epilogue: in quads, of four rows in one column for each lane.  Register r of quad (i,j) of a wave tile holds
  //      row  16*i + 4*(lane/16) + r ,  column 16*j + lane%16  (blocks of 32 x 32: row 32*(i/2) + 8*(2*(i%2) + j%2) + 4*(lane/32) + r,
  //      column 32*(j/2) + lane%32) ----
  // Fused loss: the bf16 target tile is first copied into the (now idle) LDS tile buffers with
  // coalesced 16-byte loads, then every lane picks its own elements from LDS.  Differences and
  // squares are formed in fp32, summed over the 16 registers of four quads in fp32, and
  // every such partial is added in fp64 (the loss difference of the two passes is ~1e-6 of the
  // loss, far below fp32 resolution of a long sum).
  // K in two parts: either part keeps half of the row blocks and gets the other's sums of them through the second part's tile
  // buffers (idle by now).  The first part's sum is added to the second's.
  constexpr int QM = 2 * WMB, QN = 2 * WNB, KB = QM / KS;       // quads of a wave; KB: its rows of them in the epilogue
  auto quad = [&](int i, int j) {
    if constexpr (BLK == 16) {
      return acc[i][j];
    } else {
      const float16_t b = acc[i / 2][j / 2];
      const int r = 8 * (i % 2) + 4 * (j % 2);
      return float4_t{b[r], b[r + 1], b[r + 2], b[r + 3]};
    }
  };
  float4_t out[KB][QN];
  if constexpr (KS == 1) {
#pragma unroll
    for (int i = 0; i < KB; ++i)
#pragma unroll
      for (int j = 0; j < QN; ++j) out[i][j] = quad(i, j);
  } else {
    float4_t* const given = reinterpret_cast<float4_t*>(smem + tiled_lds_bytes(BM, BN) / 2) + (size_t)wave * (QM * QN * 64) + lane;
    __syncthreads();                              // every wave is done with the tile buffers
#pragma unroll
    for (int i = 0; i < KB; ++i)
#pragma unroll
      for (int j = 0; j < QN; ++j) given[(kpart * KB * QN + i * QN + j) * 64] = kpart ? quad(i, j) : quad(i + KB, j);
    __syncthreads();
#pragma unroll
    for (int i = 0; i < KB; ++i)
#pragma unroll
      for (int j = 0; j < QN; ++j) out[i][j] = (kpart ? quad(i + KB, j) : quad(i, j)) + given[((1 - kpart) * KB * QN + i * QN + j) * 64];
  }
  constexpr int TROW = TN * 2 + 32;               // LDS row stride of the target tile in bytes
  const FwdParams pe = cold();
  bool staged = false;
  if (FUSE_LOSS) {
    staged = ((pe.N & 7) == 0) && ((reinterpret_cast<uintptr_t>(pe.target) & 15) == 0);
    if (staged) {
      constexpr int CPR = TN / 8;                 // 16-byte chunks per tile row
      constexpr int ROWS_PER_PASS = 64 * NWAVES * KS / CPR;
      uint8_t* const T = reinterpret_cast<uint8_t*>(smem);
      const int c = tid % CPR, r0 = tid / CPR;
      __syncthreads();                            // every wave is done with the tile buffers
      // The loads of a batch are issued before the first one is used: guarded loads in a loop would each
      // be waited for before the next is issued (16 memory round trips in a row).  Batches of four:
      // on the full stack larger bursts measured slower (8 at a time: +3 % step time), presumably because
      // they delay the operand loads of the neighbouring workgroups' main loops.  Rows and columns past
      // the matrix re-read its last row / last 8 columns; those LDS entries are never looked at.
      constexpr int PASSES = BM / ROWS_PER_PASS, BATCH = 4;
      static_assert(PASSES % BATCH == 0, "whole batches");
      const int ncl = min(n0 + 8 * c, pe.N - 8);
#pragma unroll
      for (int b = 0; b < PASSES; b += BATCH) {
        u32x4 t[BATCH];
#pragma unroll
        for (int i = 0; i < BATCH; ++i) {
          const int m = min(m0 + r0 + ROWS_PER_PASS * (b + i), pe.M - 1);
          t[i] = *reinterpret_cast<global_u32x4>(pe.target + (size_t)m * pe.N + ncl);
        }
#pragma unroll
        for (int i = 0; i < BATCH; ++i)
          *reinterpret_cast<u32x4*>(T + (r0 + ROWS_PER_PASS * (b + i)) * TROW + 16 * c) = t[i];
      }
      __syncthreads();
    }
  }
  double loss = 0.0;
  // Element (i, j, r) of this lane, r < 16: register r%4 of quad (2 i + r/8, 2 j + r/4 % 2), tile row ml0 + row_of(i, r), tile column
  // nl0 + column_of(j, r).
  // DUAL: the waves of the second half of a wave row hold the -eps forward of the same columns.
  const int wn_col = DUAL ? wn % (WAVES_N / 2) : wn;
  const int mw = wm * 32 * WMB + 16 * KB * kpart, nw = wn_col * 32 * WNB, ml0 = mw + 4 * (lane >> LANE_SHIFT), nl0 = nw + (lane & (BLK - 1));
  auto row_of = [](int i, int r) { return 32 * i + (BLK == 16 ? 16 * (r >> 3) : 8 * (r >> 2)) + (r & 3); };
  auto column_of = [](int j, int r) { return 32 * j + (BLK == 16 ? 16 * ((r >> 2) & 1) : 0); };
  const uint8_t* const trow = reinterpret_cast<const uint8_t*>(smem) + ml0 * TROW + nl0 * 2;
  // A quad's rows of y are pieces of 16 elements.  Where rows begin at odd multiples of four or eight bytes a piece shares its first and
  // last sector of memory with its neighbours, and two quads side by side trade rows first, so that an instruction writes two rows of 32
  // elements and not four of 16.  us of a forward, four rows -> two: 2077 x 256 at 1763 tokens 10.2 -> 9.7, 4097 x 256 at 4000 29.5 -> 28.3,
  // 16381 x 640 at 4000 111 -> 105, 11009 x 1024 at 8000 233 -> 219.  With rows at multiples of 16 bytes the trade costs: 4100 x 256 at 4000
  // 28.3 -> 28.6, 4104 x 256 28.6 -> 29.3, 4096 x 1024 at 1280 22.4 -> 22.8.
  enum { NO_Y, QUAD_ROWS, TRADED_ROWS };
  const bool trade = BLK == 16 && ((pe.N & 3) != 0 || (reinterpret_cast<uintptr_t>(pe.y) & 15) != 0);
  // FULL: whole tile inside the matrix (no bounds checks).  STAGED: targets come from LDS.
  // STORE: how y is written.  The three are compile-time so that the common cases are straight code.
  auto finish = [&](auto full_tag, auto staged_tag, auto store_tag) {
    constexpr bool FULL = decltype(full_tag)::value, STAGED = decltype(staged_tag)::value;
    constexpr int STORE = decltype(store_tag)::value;
    const uint32_t ybase = (uint32_t)(m0 + ml0) * (uint32_t)pe.N + (uint32_t)(n0 + nl0);   // M*N < 2^32 checked on the host
    if constexpr (STORE == TRADED_ROWS) {
      // register h of a traded pair: row 16*i + 8*(lane/32) + 4*h + r, column 32*j + lane%32
      const int mt = m0 + mw + 8 * (lane >> 5), nt = n0 + nw + (lane & 31);
      const uint32_t tbase = (uint32_t)mt * (uint32_t)pe.N + (uint32_t)nt;
#pragma unroll
      for (int i = 0; i < KB; ++i)
#pragma unroll
        for (int j = 0; j < WNB; ++j)
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            const auto rows = __builtin_amdgcn_permlane16_swap(__float_as_uint(out[i][2 * j][r]), __float_as_uint(out[i][2 * j + 1][r]), false, false);
#pragma unroll
            for (int h = 0; h < 2; ++h) {
              const int dm = 16 * i + 4 * h + r, dn = 32 * j;
              if (FULL || (mt + dm < pe.M && nt + dn < pe.N)) pe.y[tbase + (uint32_t)dm * (uint32_t)pe.N + (uint32_t)dn] = __uint_as_float(rows[h]);
            }
          }
    }
#pragma unroll
    for (int i = 0; i < WMB / KS; ++i) {
#pragma unroll
      for (int j = 0; j < WNB; ++j) {
        float part = 0.0f;
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const int dm = row_of(i, r), dn = column_of(j, r);
          if (FULL || (m0 + ml0 + dm < pe.M && n0 + nl0 + dn < pe.N)) {
            const float v = out[2 * i + (r >> 3)][2 * j + ((r >> 2) & 1)][r & 3];
            const uint32_t off = ybase + (uint32_t)dm * (uint32_t)pe.N + (uint32_t)dn;
            if (STORE == QUAD_ROWS) pe.y[off] = v;
            if (FUSE_LOSS) {
              uint32_t tb;
              if (STAGED) tb = *reinterpret_cast<const uint16_t*>(trow + dm * TROW + dn * 2);
              else tb = pe.target[off];
              const float d = v - __uint_as_float(tb << 16);
              part = fmaf(d, d, part);
            }
          }
        }
        loss += (double)part;
      }
    }
  };
  {
    using T = std::true_type;
    using F = std::false_type;
    const bool full = m0 + BM <= pe.M && n0 + TN <= pe.N;
    auto with_y = [&](auto full_tag, auto staged_tag) {
      if constexpr (BLK == 16) {
        if (trade) return finish(full_tag, staged_tag, std::integral_constant<int, TRADED_ROWS>{});
      }
      finish(full_tag, staged_tag, std::integral_constant<int, QUAD_ROWS>{});
    };
    using NoY = std::integral_constant<int, NO_Y>;
    if constexpr (GROUPED) {
      if (full && staged) finish(T{}, T{}, NoY{});
      else if (staged) finish(F{}, T{}, NoY{});
      else finish(F{}, F{}, NoY{});
    } else if (FUSE_LOSS) {
      if (full && staged && !pe.y) finish(T{}, T{}, NoY{});          // the step's path
      else if (staged) { if (pe.y) with_y(F{}, T{}); else finish(F{}, T{}, NoY{}); }
      else { if (pe.y) with_y(F{}, F{}); else finish(F{}, F{}, NoY{}); }
    } else {
      if (full) with_y(T{}, F{});
      else with_y(F{}, F{});
    }
  }
  if (FUSE_LOSS) {
    // One scaled partial per workgroup, plain store: a later kernel on the same stream adds them
    // up in index order, so the kernel boundary is the only synchronisation needed.
    __shared__ double wave_part[NWAVES * KS];
    const double w = wave_sum(loss);
    if (lane == 0) wave_part[any_wave] = w;
    __syncthreads();
    if (tid == 0) {
      double b = 0.0, b_minus = 0.0;
#pragma unroll
      for (int i = 0; i < NWAVES * KS; ++i) {
        if (DUAL && (i % WAVES_N) >= WAVES_N / 2) b_minus += wave_part[i];
        else b += wave_part[i];
      }
      pe.partials[bm * pe.grid_n + bn] = b * pe.loss_scale;       // indexed by tile: the sum does not depend on the launch order
      if (DUAL) pe.partials_minus[bm * pe.grid_n + bn] = b_minus * pe.loss_scale;
    }
  }
}

template <int WAVES_M, int WAVES_N, int WMB, int WNB, int DT, bool FUSE_LOSS, int FMT, int KS, int BLK>
__global__ void __launch_bounds__(64 * WAVES_M * WAVES_N * KS) linear_fwd_kernel(FwdParams p) {
  int bm, bn;
  tile_of_logical(logical_block((int)blockIdx.x, p.grid_m * p.grid_n), p.grid_m, p.grid_n, 4, bm, bn);
  linear_fwd_body<WAVES_M, WAVES_N, WMB, WNB, DT, FUSE_LOSS, FMT, false, KS, BLK>(p, bm, bn);
}

// Grouped launch: every forward of a step (all matrices, both signs) in one grid, so that the only
// partly filled round of workgroups is the last one of the step, not the last one of every matrix.
// The table (see forward_table) holds one FwdParams per MATRIX, ordered by first_block; a workgroup finds its entry by
// binary search and reads it through the constant address space (scalar loads into scalar registers).
// An entry has 2 * grid_m * grid_n workgroups: neighbouring logical ids are the +eps and the -eps
// forward of the same tile, and pairs walk the grid in strips of 2 row blocks, so the 32 workgroups
// resident on an XCD are 2 x 8 tiles x 2 signs: both forwards of a tile read the same activations and
// the same codes while those are in that XCD's L2, instead of the second forward fetching everything
// again later.  Workgroups between an entry's last tile and the next multiple of 8 have nothing to do.
// With DUAL an entry has grid_m * grid_n workgroups, each computing both forwards of a tile of half the
// width (see linear_fwd_body); the 32 workgroups resident on an XCD are then 2 x 16 such tiles.
template <int WAVES_M, int WAVES_N, int WMB, int WNB, int DT, bool FUSE_LOSS, int FMT, bool DUAL = false, int BLK = 16, int SHARED = kNotShared>
__global__ void __launch_bounds__(64 * WAVES_M * WAVES_N) linear_fwd_table_kernel(const FwdParams* table, int n_entries, InlineForwards) {
  constexpr int W = (int)(sizeof(FwdParams) / 4), FB = (int)(offsetof(FwdParams, first_block) / 4);
  static_assert(sizeof(FwdParams) % 4 == 0 && offsetof(FwdParams, first_block) % 4 == 0, "table entry is read as words");
  const table_words tab = forward_table(table);
  int lo = 0, hi = n_entries - 1;                           // last entry whose first_block <= blockIdx.x
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if ((int)tab[mid * W + FB] <= (int)blockIdx.x) lo = mid; else hi = mid - 1;
  }
  struct Words { uint32_t w[W]; } raw;
#pragma unroll
  for (int i = 0; i < W; ++i) raw.w[i] = tab[lo * W + i];
  FwdParams p = __builtin_bit_cast(FwdParams, raw);
  const int bid = (int)blockIdx.x - p.first_block, count = (DUAL || SHARED ? 1 : 2) * p.grid_m * p.grid_n;
  if (bid >= count) return;
  const int L = logical_block(bid, count);
  int bm, bn;
  if (DUAL || SHARED) {
    tile_of_logical(L, p.grid_m, p.grid_n, 2, bm, bn);
  } else {
    tile_of_logical(L >> 1, p.grid_m, p.grid_n, 2, bm, bn);
    if (L & 1) {                                            // the -eps forward of the tile
      p.x = p.x_minus;
      p.partials = p.partials_minus;
      p.signed_eps = -p.signed_eps;
    }
  }
  linear_fwd_body<WAVES_M, WAVES_N, WMB, WNB, DT, FUSE_LOSS, FMT, DUAL, 1, BLK, true, SHARED>(p, bm, bn, tab + lo * W);
}

// ---- host side -----------------------------------------------------------------------------

static int g_tile_config = 0;      // 0 = choose by shape, 1 = 128x128 (4 waves, K whole, the blocks of the grouped launch), 2 = 256x256 (8 waves), 3 = 2 + always group the step,
                                   // 4, 5 = as 0 with the few-token path's 32- / 48-row passes forced (see small_m_force_rblocks),
                                   // 6 = as 0 + always group the step, 7 = as 0 + non-temporal code stream in every one-slice launch,
                                   // 8, 9 = as 0 with the few-token path's split kernel always / never chosen, 10 = 9 and 7,
                                   // 11 = the one-dense-pass kernel wherever it can run (chosen by shape with 0, never with the others),
                                   // 12 = the tiled kernel with one dense product wherever it can run (likewise)
static bool few_token_enabled() { return g_tile_config == 0 || g_tile_config >= 4; }

static int ilog2_exact(int v) {
  int s = 0;
  while ((1 << s) < v) ++s;
  return (1 << s) == v ? s : -1;
}

static int validate_desc(const szo_linear_desc* d, int sign, bool need_y, bool need_target) {
  if (!d) return SZO_EINVAL;
  if (d->M < 0 || d->N < 0 || d->K <= 0 || d->nnz < 0) return SZO_EINVAL;
  if (sign < -1 || sign > 1) return SZO_EINVAL;
  if (d->tile_dtype != SZO_TILE_F16 && d->tile_dtype != SZO_TILE_BF16) return SZO_EINVAL;
  if (d->format != SZO_FORMAT_UNIFORM && d->format != SZO_FORMAT_LUT) return SZO_EINVAL;
  const bool table_format = d->format == SZO_FORMAT_LUT;
  if (!table_format && (d->group <= 0 || d->K % d->group)) return SZO_EINVAL;
  if (d->nnz_base & 3) return SZO_EINVAL;
  if (!table_format && d->group != 32 && d->group != 64 && d->group != 128) return SZO_EUNSUPPORTED;
  if (table_format && d->tile_dtype != SZO_TILE_F16) return SZO_EUNSUPPORTED;
  if (d->K % BK) return SZO_EUNSUPPORTED;
  if ((uint64_t)d->N * (uint64_t)d->K > 0xFFFFFFFFull) return SZO_EUNSUPPORTED;
  if (d->M > 0x7FFFFFFF || d->N > 0x7FFFFFFF || d->nnz > 0xFFFFFFFFll) return SZO_EUNSUPPORTED;
  if ((uint64_t)d->M * (uint64_t)d->N > 0xFFFFFFFFull) return SZO_EUNSUPPORTED;
  if (d->M == 0 || d->N == 0) return SZO_OK;
  if (!d->x || !d->qweight || !d->tile_ptr) return SZO_EINVAL;
  if (table_format ? (!d->lut || ((uintptr_t)d->lut & 15)) : !d->scales) return SZO_EINVAL;
  if (d->nnz > 0 && (!d->sp_idx || !d->sp_val)) return SZO_EINVAL;
  if (need_y && !d->y) return SZO_EINVAL;
  if (need_target && !d->target) return SZO_EINVAL;
  if (((uintptr_t)d->x & 15) || ((uintptr_t)d->x_minus & 15) || ((uintptr_t)d->qweight & 15) || ((uintptr_t)d->scales & 1) ||
      ((uintptr_t)d->tile_ptr & 3) || ((uintptr_t)d->sp_idx & 15) || ((uintptr_t)d->sp_val & 15) ||
      ((uintptr_t)d->y & 3) || ((uintptr_t)d->target & 1))
    return SZO_EINVAL;
  return SZO_OK;
}

template <int WAVES_M, int WAVES_N, int WMB, int WNB, int DT, bool FUSE, int FMT = SZO_FORMAT_UNIFORM, int KS = 1, int BLK = 16>
static int launch(FwdParams& p, hipStream_t stream) {
  constexpr int BM = 32 * WMB * WAVES_M, BN = 32 * WNB * WAVES_N;
  p.grid_m = (p.M + BM - 1) / BM;
  p.grid_n = (p.N + BN - 1) / BN;
  const int64_t blocks = (int64_t)p.grid_m * p.grid_n;
  if (blocks > 0x7FFFFFFF) return SZO_EUNSUPPORTED;
  constexpr size_t main_bytes = KS * (size_t)tiled_lds_bytes(BM, BN);
  constexpr size_t target_bytes = FUSE ? (size_t)BM * (BN * 2 + 32) : 0;      // staged target tile of the fused loss
  constexpr size_t lds_bytes = main_bytes > target_bytes ? main_bytes : target_bytes;
  auto kern = linear_fwd_kernel<WAVES_M, WAVES_N, WMB, WNB, DT, FUSE, FMT, KS, BLK>;
  static std::atomic<uint64_t> lds_limit_set{0};     // per instantiation
  int rc = set_lds_limit_once(lds_limit_set, (const void*)kern, lds_bytes);
  if (rc != SZO_OK) return rc;
  rc = timing_begin(stream);
  if (rc != SZO_OK) return rc;
  kern<<<(unsigned)blocks, 64 * WAVES_M * WAVES_N * KS, lds_bytes, stream>>>(p);
  SZO_LAUNCH_CHECK();
  return timing_end(stream);
}

// Which workgroup tile a shape runs with, and how many workgroups (= loss partials) that makes.
static int plan_tiles(int M, int N, int format, int* blocks_out) {
  int cfg = g_tile_config >= 4 ? 0 : g_tile_config;
  if (format == SZO_FORMAT_LUT) cfg = 2;          // the table format exists for the 256x256 tile only
  if (cfg == 0) {
    const int64_t big_blocks = (int64_t)((M + 255) / 256) * ((N + 255) / 256);
    cfg = big_blocks >= 192 ? 2 : 1;
  }
  if (cfg == 3) cfg = 2;
  const int t = cfg == 2 ? 256 : 128;
  const int64_t blocks = (int64_t)((M + t - 1) / t) * ((N + t - 1) / t);
  *blocks_out = blocks > 0x7FFFFFFF ? -1 : (int)blocks;
  return cfg;
}

// 128 x 128 tiles, K whole: blocks of 32 x 32, half as many matrix instructions, where a weight wave's instructions bound the launch, of
// 16 x 16 where power does.  With the bf16 tile, whose dequantisation is longest, always.  With the fp16 tile while few CUs have more than one
// tile, a little further with denser masks, and for short K with unaligned rows of y, which blocks of 32 x 32 store in two rows of 32
// by themselves.  us, 16x16x32 -> 32x32x16: bf16 forwards of 8192 x 8192 at 700 tokens 181.5 -> 173.9, 4096 x 4096 at 1280 / 2000 93.4 / 94.9 ->
// 88.7 / 93.4, a step over 8192 x 4096 at 700 and 0.8 % 218 -> 210; fp16 forwards of 4096 x 4096 at 1100 / 1280 (288 / 320 tiles) 69.0 / 68.7 -> 66.7 /
// 67.0, 4096 x 11008 at 1200 174.9 -> 168.0, 4096 x 4160 at 500 (128 tiles) 51.9 -> 50.4; beyond the line 4096 x 4096 at 1400 (352) 69.4 -> 70.4 and
// 69.8 -> 68.9 on two machines, at 1500 / 2000 (384 / 512) 70.2 / 77.7 -> 70.7 / 81.2; with 0.3 / 0.5 / 1 % at 1500 72.0 / 73.0 / 77.3 -> 71.4 / 72.2 / 75.6, a
// step over 8192 x 8192 at 700 and 0.5 % 301 -> 290; 5003 x 256 / 1024 at 1100 (360) 11.6 / 23.1 -> 11.4 / 22.6, 3333 x 256 / 1024 / 2048 at 2000 (432)
// 12.1 / 23.9 / 39.6 -> 11.8 / 24.0 / 40.3.
static bool wide_blocks(int tiles, const FwdParams& p) {
  return tiles <= 320 || (tiles <= 384 && 250ll * p.nnz >= (int64_t)p.N * p.K) || ((p.N & 3) != 0 && p.K <= 1024);
}

// Tables (256 x 256 tiles): up to this many a K step is bound by the look-ups and blocks of 32 x 32 are faster, with more of the chip at work
// power decides.  us of a forward of 4096 x 4096, 32x32x16 / 16x16x32, at 1024 / 2048 / 2560 / 2816 / 3072 / 4096 tokens (64 / 128 / 160 / 176 / 192 /
// 256 tiles) 86 / 96, 88 / 97, 96 / 99, 101.1 / 101.0, 106 / 105, 131 / 126; beyond a round at 5120 / 8192 209 / 211, 257 / 250; 1024
// columns at 2304 / 3072 30.5 / 31.7, 34.9 / 34.4; a step over a Llama block with outputs at 600 1583 / 1766.
constexpr int kFewTableTiles = 168;

template <int DT, bool FUSE>
static int dispatch_tile(FwdParams& p, hipStream_t stream) {
  int blocks;
  if (plan_tiles(p.M, p.N, SZO_FORMAT_UNIFORM, &blocks) == 2) return launch<2, 4, 4, 2, DT, FUSE>(p, stream);
  const bool chosen = g_tile_config == 0 || g_tile_config >= 4;
  if (chosen && tiles_halve_k(blocks, p.K)) return launch<2, 2, 2, 2, DT, FUSE, SZO_FORMAT_UNIFORM, 2>(p, stream);
  if (DT == SZO_TILE_BF16 || (chosen && wide_blocks(blocks, p))) return launch<2, 2, 2, 2, DT, FUSE, SZO_FORMAT_UNIFORM, 1, 32>(p, stream);
  return launch<2, 2, 2, 2, SZO_TILE_F16, FUSE>(p, stream);
}

// Enqueues one forward.  With `partials` set the loss is fused: workgroup b stores
// scale * sum (y - target)^2 of its tile to partials[b].
int fill_params(FwdParams& p, const szo_linear_desc* d, uint64_t seed, uint64_t step, int sign, float eps,
                double* partials, double scale) {
  p = FwdParams{};
  p.x = (global_u16)d->x;
  p.qweight = (global_u8)d->qweight;
  p.scales = (global_u16)d->scales;
  p.lut = (global_u16)d->lut;
  p.tile_ptr = (global_u32)d->tile_ptr;
  p.sp_idx = (global_u32)d->sp_idx;
  p.sp_val = (global_f32)d->sp_val;
  p.y = (global_f32_out)d->y;
  p.target = (global_u16)d->target;
  p.M = (int)d->M; p.N = (int)d->N; p.K = (int)d->K;
  p.nnz = (uint32_t)d->nnz;
  p.group_shift = d->format == SZO_FORMAT_LUT ? 0 : ilog2_exact(d->group);
  p.ktiles = p.K / BK;
  p.bands = (p.N + SZO_TILE_ROWS - 1) / SZO_TILE_ROWS;
  {
    // multiplier for floor(v / K), v < 2^32: l = ceil(log2 K), mul = floor(2^32 (2^l - K) / K) + 1
    int l = 0;
    while ((1ull << l) < (uint64_t)p.K) ++l;
    if (l == 0) return SZO_EUNSUPPORTED;
    p.div_mul = (uint32_t)((((1ull << l) - (uint64_t)p.K) << 32) / (uint64_t)p.K + 1ull);
    p.div_shift = l - 1;
  }
  p.nnz_base = d->nnz_base; p.seed = seed; p.step = step;
  p.signed_eps = (float)sign * eps;
  p.partials = (global_f64_out)partials;
  p.loss_scale = scale;
  return SZO_OK;
}

// `step_minus`: this is the -eps forward of a whole step, which reads desc->x_minus where that is set.
static int run_forward(const szo_linear_desc* d, uint64_t seed, uint64_t step, int sign, float eps,
                       double* partials, double scale, hipStream_t stream, bool step_minus = false) {
  const bool fuse = partials != nullptr;
  if (d->M == 0 || d->N == 0) return SZO_OK;
  FwdParams p;
  const int frc = fill_params(p, d, seed, step, sign, eps, partials, scale);
  if (frc != SZO_OK) return frc;
  if (step_minus && d->x_minus) p.x = (global_u16)d->x_minus;
  if (d->format == SZO_FORMAT_LUT) {
    int blocks;
    plan_tiles(p.M, p.N, SZO_FORMAT_LUT, &blocks);
    if ((g_tile_config == 0 || g_tile_config >= 4) && blocks <= kFewTableTiles)
      return fuse ? launch<2, 4, 4, 2, SZO_TILE_F16, true, SZO_FORMAT_LUT, 1, 32>(p, stream)
                  : launch<2, 4, 4, 2, SZO_TILE_F16, false, SZO_FORMAT_LUT, 1, 32>(p, stream);
    return fuse ? launch<2, 4, 4, 2, SZO_TILE_F16, true, SZO_FORMAT_LUT>(p, stream)
                : launch<2, 4, 4, 2, SZO_TILE_F16, false, SZO_FORMAT_LUT>(p, stream);
  }
  if (d->tile_dtype == SZO_TILE_F16)
    return fuse ? dispatch_tile<SZO_TILE_F16, true>(p, stream) : dispatch_tile<SZO_TILE_F16, false>(p, stream);
  return fuse ? dispatch_tile<SZO_TILE_BF16, true>(p, stream) : dispatch_tile<SZO_TILE_BF16, false>(p, stream);
}

// The sparse update of a step: one grouped launch for the whole stack (per-matrix launches when the table does not fit).
// With partials_per_sign > 0 g is formed from that many loss partials first; otherwise scalars[2] holds it.
static int update_all(const szo_linear_desc* descs, int n, uint64_t seed, uint64_t step, float eps, float lr, double* scalars,
                      double* partials, int64_t partials_per_sign, void* table_dev, hipStream_t s) {
  if (n <= (table_dev ? kMaxStepMatrices : kInlineMats) && small_m_table_bytes(n) <= kTableBytesPerMatrix * (size_t)kMaxStepMatrices)
    return small_m_step(descs, n, seed, step, eps, lr, table_dev, partials, partials_per_sign, scalars, false, s);
  if (partials_per_sign > 0) {
    const int rc = reduce_step(partials, (int)partials_per_sign, eps, scalars, s);
    if (rc != SZO_OK) return rc;
  }
  for (int i = 0; i < n; ++i) {
    const int rc = szo_sparse_update(descs[i].sp_val, descs[i].sp_idx, descs[i].nnz, descs[i].nnz_base, seed, step,
                                     scalars + 2, lr, s);
    if (rc != SZO_OK) return rc;
  }
  return SZO_OK;
}

static double* partial_area(void* workspace) { return (double*)((char*)workspace + kWorkspaceHeader); }
static void* copy_area(void* workspace) { return (void*)(((uintptr_t)workspace + kWorkspaceCopyOffset + 127) & ~(uintptr_t)127); }

template <int DT, int FMT = SZO_FORMAT_UNIFORM, int TILE = 256, bool DUAL = false, int SHARED = kNotShared>
static int launch_table(const ForwardTableArgs& t, int64_t blocks, hipStream_t stream) {
  static_assert(TILE == 256 || TILE == 128, "two workgroup tiles exist");
  constexpr int BM = TILE, BN = TILE;
  constexpr int WAVES_N = TILE == 256 ? 4 : 2, WMB = TILE == 256 ? 4 : 2;      // 2x4 waves of 128x64, or 2x2 of 64x64
  constexpr size_t main_bytes = 2 * (size_t)(BM + BN) * BK * sizeof(uint16_t) + (size_t)(BN / 64) * (kWindow * 6 + 128);
  constexpr size_t target_bytes = (size_t)BM * (BN * 2 + 32);
  constexpr size_t lds_bytes = SHARED ? (size_t)SharedLds::BYTES : main_bytes > target_bytes ? main_bytes : target_bytes;
  static_assert(lds_bytes >= main_bytes, "the sensitive product's buffers replace the operands");
  constexpr int BLK = TILE == 128 && DT == SZO_TILE_BF16 ? 32 : 16;            // as in dispatch_tile
  auto kern = linear_fwd_table_kernel<2, WAVES_N, WMB, 2, DT, true, FMT, DUAL, BLK, SHARED>;
  static std::atomic<uint64_t> lds_limit_set{0};
  int rc = set_lds_limit_once(lds_limit_set, (const void*)kern, lds_bytes);
  if (rc != SZO_OK) return rc;
  if (!SHARED) rc = timing_begin(stream);                   // SHARED: its caller times the copies too
  if (rc != SZO_OK) return rc;
  kern<<<(unsigned)blocks, 128 * WAVES_N, lds_bytes, stream>>>(t.table, t.n_entries, t.inl);
  SZO_LAUNCH_CHECK();
  return SHARED ? SZO_OK : timing_end(stream);
}

// Both forwards of every matrix of a step as ONE launch with the loss fused: 256x256 tiles, or 128x128
// when the library chooses the tiles and no matrix has more than 128 tokens (a 256-row tile would then
// be at least half padding).
// Returns SZO_EUNSUPPORTED when the stack does not qualify (the caller then launches per matrix):
// mixed tile types or formats, a table that does not fit the workspace, or too few tiles to fill the chip.
// On success *partials_per_sign is the number of loss partials of one sign: the "+" partials are
// partials[0 .. T), the "-" partials partials[T .. 2T).
static int grouped_forwards(const szo_linear_desc* descs, int n, uint64_t seed, uint64_t step, float eps,
                            void* table_dev, double* partials, int64_t* partials_per_sign, hipStream_t stream) {
  if (g_tile_config == 1) return SZO_EUNSUPPORTED;
  int64_t max_m = 0;
  for (int i = 0; i < n; ++i) max_m = std::max<int64_t>(max_m, descs[i].N > 0 ? descs[i].M : 0);
  const bool auto_tiles = g_tile_config == 0 || g_tile_config >= 4;
  const int tile = (auto_tiles && n > 0 && descs[0].format == SZO_FORMAT_UNIFORM && max_m <= 128) ? 128 : 256;
  // Dual-sign tiles (one workgroup computes both forwards of 256 x 128 outputs and dequantises the weights
  // once for both) when the library chooses the tiles and no layer has a second activation set.
  bool dual = auto_tiles && tile == 256 && n > 0 && descs[0].format == SZO_FORMAT_UNIFORM;
  for (int i = 0; dual && i < n; ++i) dual = descs[i].x_minus == nullptr;
  const int tile_n = dual ? tile / 2 : tile;
  int64_t T = 0, wgs = 0;          // loss partials per sign; workgroups of the launch
  int live = 0;
  for (int i = 0; i < n; ++i) {
    const szo_linear_desc* d = &descs[i];
    if (d->M == 0 || d->N == 0) continue;
    if (d->tile_dtype != descs[0].tile_dtype || d->format != descs[0].format) return SZO_EUNSUPPORTED;
    const int64_t t = (int64_t)((d->M + tile - 1) / tile) * ((d->N + tile_n - 1) / tile_n);
    T += t;
    wgs += dual ? t : 2 * t;
    ++live;
  }
  if ((wgs < 384 && g_tile_config != 3 && g_tile_config != 6) || T == 0 || 2 * T > kMaxLossPartials) return SZO_EUNSUPPORTED;
  if (sizeof(FwdParams) * (size_t)live > kTableBytesPerMatrix * (size_t)kMaxStepMatrices) return SZO_EUNSUPPORTED;
  static thread_local std::vector<FwdParams> table;
  table.clear();
  int64_t first_block = 0, offset = 0;
  // Half-empty last rows of tiles, which take about half as long, get entries of their own: a layer that begins there.
  const bool ordered = wgs <= 8192;
  const bool split = ordered && !dual && descs[0].format == SZO_FORMAT_UNIFORM &&
                     2 * sizeof(FwdParams) * (size_t)live <= kTableBytesPerMatrix * (size_t)kMaxStepMatrices;
  for (int i = 0; i < n; ++i) {                             // partials in the layers' order, whatever order the launch takes
    const szo_linear_desc* d = &descs[i];
    if (d->M == 0 || d->N == 0) continue;
    const double scale = 1.0 / ((double)d->M * (double)d->N);
    const int gm = (int)((d->M + tile - 1) / tile), gn = (int)((d->N + tile_n - 1) / tile_n);
    FwdParams p;
    const int rc = fill_params(p, d, seed, step, +1, eps, partials + offset, scale);
    if (rc != SZO_OK) return rc;
    p.x_minus = d->x_minus ? (global_u16)d->x_minus : p.x;
    p.partials_minus = (global_f64_out)(partials + T + offset);
    p.grid_m = gm; p.grid_n = gn;
    p.y = nullptr;                                          // the step's fused path never writes y
    const bool half = split && gm * tile - (int)d->M >= tile / 2;
    if (half && gm > 1) {
      FwdParams last = p;
      const size_t rows = (size_t)(gm - 1) * (size_t)tile;
      last.x += rows * (size_t)d->K;
      last.x_minus += rows * (size_t)d->K;
      last.target += rows * (size_t)d->N;
      last.M -= (int)rows;
      last.partials += (size_t)(gm - 1) * (size_t)gn;
      last.partials_minus += (size_t)(gm - 1) * (size_t)gn;
      last.grid_m = 1;
      table.push_back(last);
      p.M = (int)rows;
      p.grid_m = gm - 1;
    }
    table.push_back(p);
    offset += (int64_t)gm * gn;
  }
  // Longest K first, so that the launch ends with its shortest tiles: a tile's time is its walk along K, one tile per CU at a
  // time.  In the caller's order it ended with the last block's longest layer: two Mistral blocks with two sets of activations at
  // 333 tokens (1344 tiles, the last 64 of them 3.4 times as long as the others) 889 -> 812 us per step.  From 32 rounds of
  // workgroups on there is nothing to gain (a Mistral block at 8192 tokens, 42 rounds, 6251 -> 6295): the caller's order.
  // Half-empty tiles are ordered by half their K: those blocks 733 -> 688 on another machine, one OPT / Mistral block at 600 tokens
  // 575 / 619 -> 517 / 541, two Llama blocks at 850 1479 -> 1448.
  if (ordered) {
    auto walk = [&](const FwdParams& p) { return (int64_t)p.K * (split && p.grid_m * tile - p.M >= tile / 2 ? 1 : 2); };
    std::stable_sort(table.begin(), table.end(), [&](const FwdParams& a, const FwdParams& b) { return walk(a) > walk(b); });
  }
  for (FwdParams& p : table) {
    p.first_block = (int)first_block;
    first_block += ((dual ? 1 : 2) * (int64_t)p.grid_m * p.grid_n + 7) & ~(int64_t)7;
    if (first_block > 0x7FFFFFFF) return SZO_EUNSUPPORTED;
  }
  static thread_local ForwardTableArgs t;
  int rc = place_table(table.data(), table.size(), table_dev, stream, t);
  if (rc != SZO_OK) return rc;
  *partials_per_sign = T;
  if (descs[0].format == SZO_FORMAT_LUT)
    return launch_table<SZO_TILE_F16, SZO_FORMAT_LUT>(t, first_block, stream);
  if (tile == 128) {
    if (descs[0].tile_dtype == SZO_TILE_F16)
      return launch_table<SZO_TILE_F16, SZO_FORMAT_UNIFORM, 128>(t, first_block, stream);
    return launch_table<SZO_TILE_BF16, SZO_FORMAT_UNIFORM, 128>(t, first_block, stream);
  }
  if (dual) {
    if (descs[0].tile_dtype == SZO_TILE_F16)
      return launch_table<SZO_TILE_F16, SZO_FORMAT_UNIFORM, 256, true>(t, first_block, stream);
    return launch_table<SZO_TILE_BF16, SZO_FORMAT_UNIFORM, 256, true>(t, first_block, stream);
  }
  if (descs[0].tile_dtype == SZO_TILE_F16)
    return launch_table<SZO_TILE_F16>(t, first_block, stream);
  return launch_table<SZO_TILE_BF16>(t, first_block, stream);
}

// Whether the one-dense-pass kernel rounds a layer's weights to the tile's type too (the others' scales it applies in fp32).
static bool onepass_rounds(const szo_linear_desc& d) { return d.tile_dtype == SZO_TILE_BF16 || d.group != 128; }

// Whether the dense product once for both signs, with the sensitive products behind it, is faster than two products (dual-sign tiles): what
// the second product takes against copying the activations and the sensitive products, in units of one column of K in one tile.  Fitted
// to four to eight layers of 4096 x K at 4096 tokens, us per step, two products -> one: K = 256 / 1024 / 4096 at 0.1 % 212 / 497 / 843 -> 212 / 390 / 570,
// at 0.4 % 212 / 508 / 872 -> 219 / 433 / 726, at 1 % 211 / 517 / 910 -> 238 / 610 / 1009.  The line is drawn for masks with rows full of
// entries, whose bands take longer (a Llama block with half of them in 1 % of the rows, 0.4 % / 1 %: 2668 / 2956 -> 2498 / 4204).
// Only in steps of more than 4096 tiles, 16 rounds of workgroups.  That line is not where the two cost the same: one Llama block at 4096
// tokens (2656 tiles) would take 1750 us instead of 2630.  Up to it a step keeps the single-layer calls' roundings, to whose losses a block's
// are compared at 1e-12 (tests/test_gpu_full_size.py), which a weight rounded together with its perturbation makes true and D +- eps Z does not
// (1e-9 of the loss apart).  Beyond it, two products -> here: a Mistral block at 8192 tokens and 0.01 / 0.1 / 0.4 / 0.55 % 5572 / 5623 / 5820 /
// 5866 -> 3305 / 3612 / 4545 / 4945, two Llama blocks at 4096 and 0.1 / 0.4 % 5391 / 5506 -> 3425 / 4246.
// `instead_of_onepass`: of a step that the kernel with tiles of 64 token rows takes otherwise, where that one rounds weights to the tile's type
// too (bf16 tile, groups other than 128).  From 512 tiles and tokens on, with a third of the second product to spare: bf16 tile, 0.1 %,
// there -> here: one Llama block at 1000 / 2048 tokens 626 / 1208 -> 471 / 878, four OPT blocks at 520 / 1300 1416 / 3201 -> 1208 / 2428; groups
// of 64 likewise 561 / 1082 -> 463 / 869, 1264 / 2850 -> 1201 / 2462, one Llama block with 0.3 % at 2048 1302 -> 1034.
// Fewer tiles: one OPT block at 768 tokens (432) 410 -> 446, a layer of 4096 x 4096 at 2048 (128) 96 -> 117.
static bool shared_pays(const szo_linear_desc* descs, int n, bool instead_of_onepass) {
  double tiles = 0.0, second = 0.0, here = 0.0;             // tiles: of 256 x 256 outputs, one workgroup each
  for (int i = 0; i < n; ++i) {
    const szo_linear_desc& d = descs[i];
    if (d.M == 0 || d.N == 0) continue;
    if (instead_of_onepass && (d.M <= 512 || !onepass_rounds(d))) return false;
    const double rows = (double)((d.M + 255) / 256), columns = (double)((d.N + 255) / 256), K = (double)d.K;
    tiles += rows * columns;
    second += rows * columns * 1.14 * K;
    here += rows * (columns * (256.0 + 160.0 * (double)d.nnz / (double)d.N) + 2.3 * K);
  }
  return instead_of_onepass ? tiles >= 512.0 && here < 0.65 * second : tiles > 4096.0 && here < second;
}

// The launches of a step with one dense product: each of as many layers as the copy area has room for the activations of.
struct SharedPlan {
  struct Launch { size_t first, items; };                   // its first layer, the end of its copies
  std::vector<Launch> launches;
  std::vector<int> layers;                                  // those with tokens and outputs
  std::vector<size_t> copy;                                 // which copy each of them reads
  std::vector<TransposeItem> items;                         // the copies; x -> out, here an offset
  std::unordered_map<const void*, size_t> copy_of;          // the launch's latest copy of these activations
  int64_t tiles;                                            // of 256 x 256 outputs
  size_t bytes;                                             // of the copy area that is written
  bool make(const szo_linear_desc* descs, int n) {          // false if the layers do not qualify
    launches.clear();
    layers.clear();
    copy.clear();
    items.clear();
    copy_of.clear();
    tiles = 0;
    bytes = 0;
    size_t used = 0;
    for (int i = 0; i < n; ++i) {
      const szo_linear_desc& d = descs[i];
      if (d.tile_dtype != descs[0].tile_dtype || d.format != SZO_FORMAT_UNIFORM) return false;
      if (d.M == 0 || d.N == 0) continue;
      const size_t need = (size_t)((d.M + 63) / 64) * (size_t)d.K * 128;
      if (d.x_minus || d.K >= (1 << 21) || need > kCopyAreaBytes) return false;      // offsets within a tile's rows of x: 31 bits
      const auto known = copy_of.find(d.x);                 // several matrices may be applied to the same activations
      size_t c = known == copy_of.end() ? items.size() : known->second;
      if (c < items.size() && (items[c].M != (int)d.M || items[c].K != (int)d.K)) c = items.size();
      if (c == items.size() && used + need > kCopyAreaBytes) {
        copy_of.clear();
        used = 0;
      }
      if (used == 0) launches.push_back(Launch{layers.size(), 0});
      if (c == items.size()) {
        items.push_back(TransposeItem{(const uint16_t*)d.x, (uint16_t*)(uintptr_t)used, (int)d.M, (int)d.K, 0});
        used += need;
        bytes = std::max(bytes, used);
        copy_of[d.x] = c;
      }
      layers.push_back(i);
      copy.push_back(c);
      launches.back().items = items.size();
      tiles += ((d.M + 255) / 256) * ((d.N + 255) / 256);
    }
    return tiles > 0 && 2 * tiles <= kMaxLossPartials && sizeof(FwdParams) * layers.size() <= kTableBytesPerMatrix * (size_t)kMaxStepMatrices;
  }
};

// Both forwards of every matrix with the dense product computed once (szo_shared.h), the loss fused: launches of 256 x 256 tiles, each behind
// the copies of its layers' activations in the order that its sensitive products read them.
// SZO_EUNSUPPORTED, with nothing enqueued, when the stack does not qualify.
static int shared_forwards(const szo_linear_desc* descs, int n, bool instead_of_onepass, uint64_t seed, uint64_t step, float eps, void* table_dev,
                           void* copies, double* partials, int64_t* partials_per_sign, hipStream_t stream) {
  constexpr int tile = 256;
  static thread_local SharedPlan plan;
  if (!plan.make(descs, n)) return SZO_EUNSUPPORTED;        // reject everything before anything is enqueued
  const int64_t T = plan.tiles;
  const bool f16 = descs[0].tile_dtype == SZO_TILE_F16;
  // Steps that the one-dense-pass kernel would take have its sums, one by one in fp64; the others those of two products (a step of 9.1 ms
  // with rounded weights 1.3 % less).  Forced: by what tells the layers apart.
  bool fp64_sums = instead_of_onepass || g_tile_config == 12;
  for (int i : plan.layers) fp64_sums = fp64_sums && onepass_rounds(descs[i]);
  // One table for the whole step, staged once: the host runs as many steps ahead as with one launch.
  static thread_local std::vector<FwdParams> table;
  static thread_local std::vector<int64_t> blocks;          // workgroups of each launch
  table.clear();
  blocks.clear();
  for (TransposeItem& it : plan.items) it.out = (uint16_t*)((char*)copies + (uintptr_t)it.out);
  int64_t offset = 0;
  bool staged = false;
  auto end_of = [&](size_t launch) { return launch + 1 < plan.launches.size() ? plan.launches[launch + 1].first : plan.layers.size(); };
  for (size_t l = 0; l < plan.launches.size(); ++l) {
    const size_t first = plan.launches[l].first, end = end_of(l);
    const int64_t before = offset;
    for (size_t e = first; e < end; ++e) {
      const szo_linear_desc& d = descs[plan.layers[e]];
      FwdParams p;
      const int rc = fill_params(p, &d, seed, step, +1, eps, partials + offset, 1.0 / ((double)d.M * (double)d.N));
      if (rc != SZO_OK) return rc;
      p.x_minus = (global_u16)plan.items[plan.copy[e]].out;
      p.partials_minus = (global_f64_out)(partials + T + offset);
      p.grid_m = (int)((d.M + tile - 1) / tile);
      p.grid_n = (int)((d.N + tile - 1) / tile);
      p.y = nullptr;
      offset += (int64_t)p.grid_m * p.grid_n;
      table.push_back(p);
    }
    // Longest K first, as above: the launch ends with its shortest tiles.
    if (offset - before <= 8192) std::stable_sort(table.begin() + (ptrdiff_t)first, table.end(), [](const FwdParams& a, const FwdParams& b) { return a.K > b.K; });
    int64_t first_block = 0;
    for (size_t e = first; e < end; ++e) {
      table[e].first_block = (int)first_block;
      first_block += ((int64_t)table[e].grid_m * table[e].grid_n + 7) & ~(int64_t)7;      // fits: fewer than 2^20 tiles and 4096 entries
    }
    blocks.push_back(first_block);
    staged = staged || end - first > (size_t)kInlineForwards;
  }
  int rc = timing_begin(stream);
  if (rc == SZO_OK && staged) rc = stage_table(table.data(), sizeof(FwdParams) * table.size(), table_dev, stream);
  size_t item = 0;
  for (size_t l = 0; rc == SZO_OK && l < plan.launches.size(); ++l) {
    const size_t first = plan.launches[l].first, items = plan.launches[l].items;
    while (item < items) {
      TransposeArgs args;
      args.blocks = 0;
      for (args.n = 0; item < items && args.n < (int)(sizeof(args.item) / sizeof(args.item[0])); ++item) {
        TransposeItem& it = args.item[args.n++] = plan.items[item];
        it.first = args.blocks;
        args.blocks += (uint32_t)((it.M + 63) / 64) * (uint32_t)(it.K / 64);
      }
      const unsigned grid = (args.blocks + 3u) / 4u;
      if (f16) transpose_kernel<SZO_TILE_F16><<<grid, 256, 0, stream>>>(args);
      else transpose_kernel<SZO_TILE_BF16><<<grid, 256, 0, stream>>>(args);
      SZO_LAUNCH_CHECK();
    }
    static thread_local ForwardTableArgs t;
    use_table(table.data() + first, end_of(l) - first, (const FwdParams*)table_dev + first, t);
    rc = f16 ? (fp64_sums ? launch_table<SZO_TILE_F16, SZO_FORMAT_UNIFORM, 256, false, kSharedFp64Sums>(t, blocks[l], stream)
                          : launch_table<SZO_TILE_F16, SZO_FORMAT_UNIFORM, 256, false, kShared>(t, blocks[l], stream))
             : (fp64_sums ? launch_table<SZO_TILE_BF16, SZO_FORMAT_UNIFORM, 256, false, kSharedFp64Sums>(t, blocks[l], stream)
                          : launch_table<SZO_TILE_BF16, SZO_FORMAT_UNIFORM, 256, false, kShared>(t, blocks[l], stream));
  }
  if (rc != SZO_OK) return rc;
  *partials_per_sign = T;
  return timing_end(stream);
}

// Which of the ways a step may go.  A later one is taken where those before it find that they cannot: the dense product once in large tiles
// instead of in tiles of 64 token rows; those; the few-token path (up to 2^20 workgroups); once in large tiles instead of twice; twice.
struct StepRoute { bool asked_for, few_rule, few, instead_of_onepass, instead_of_two; };
static StepRoute step_route(const szo_linear_desc* descs, int n, int flags) {
  const bool fuse = (flags & SZO_STEP_FUSED_LOSS) != 0, copies = fuse && !(flags & SZO_STEP_SMALL_WORKSPACE);
  // Few-token stacks: one pass over the weights serves both forwards of the step.  SZO_STEP_ONE_DENSE_PASS: also at token counts
  // that the rule leaves to the tiled kernel.
  const bool can_few = fuse && few_token_enabled() && g_tile_config != 12 && n <= kMaxStepMatrices;
  StepRoute r;
  r.asked_for = (flags & SZO_STEP_ONE_DENSE_PASS) != 0;
  r.few_rule = can_few && small_m_eligible(descs, n, false, false, 2);
  r.few = r.few_rule || (can_few && r.asked_for && small_m_eligible(descs, n, true, false, 2));
  r.instead_of_onepass = copies && g_tile_config == 0 && shared_pays(descs, n, true) && onepass_partials(descs, n, r.few_rule, r.asked_for, false, false) > 0;
  r.instead_of_two = copies && !r.few && (g_tile_config == 12 || (g_tile_config == 0 && shared_pays(descs, n, false)));
  return r;
}

// Device address of `scratch` on the current device, looked up once per device.
static int noalloc_partials(double** out) {
  constexpr int kMaxDevices = 64;
  static std::mutex mu;
  static double* ptr[kMaxDevices] = {};
  int dev = 0;
  SZO_HIP(hipGetDevice(&dev));
  if (dev < 0 || dev >= kMaxDevices) return SZO_EUNSUPPORTED;
  std::lock_guard<std::mutex> lock(mu);
  if (!ptr[dev]) {
    void* p = nullptr;
    SZO_HIP(hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)));
    if (!p) return SZO_ELAUNCH;
    ptr[dev] = (double*)p;
  }
  *out = ptr[dev];
  return SZO_OK;
}

}  // namespace szo

using namespace szo;

extern "C" {

int szo_zo_step_noalloc(const szo_linear_desc* descs, int n, uint64_t seed, uint64_t step, float eps, float lr,
                        double* scalars, void* stream) {
  if (n < 0 || (n > 0 && !descs) || !scalars) return SZO_EINVAL;
  hipStream_t s = (hipStream_t)stream;
  // Kernel choice as in szo_zo_step: the few-token kernel (one launch per layer, both signs) when every
  // layer qualifies for it -- here also: no layer with a second activation set, which needs the grouped
  // launch's dual kernel -- else the tiled kernel, one launch per layer and sign.
  // `less`: when the partials of the layers' preferred launches exceed the array, the ones with fewer of them.
  bool few_all = false;
  Partials less = kBandsInParts;
  int64_t T = 0;
  for (Partials attempt : {kBandsInParts, kWholeBands, kStreamKernel}) {
    less = attempt;
    few_all = few_token_enabled() && small_m_eligible(descs, n, false, true, 2) && (less != kStreamKernel || small_m_eligible(descs, n, true, true, 2));
    T = 0;
    for (int i = 0; i < n; ++i) {     // reject everything before anything is enqueued
      const szo_linear_desc* d = &descs[i];
      const int rc = validate_desc(d, 1, false, true);
      if (rc != SZO_OK) return rc;
      if (d->nnz > 0 && (!d->sp_val || ((uintptr_t)d->sp_val & 15))) return SZO_EINVAL;
      if (d->M == 0 || d->N == 0) continue;
      if (few_all) { T += small_m_launch_partials(d, less); continue; }
      int blocks;
      plan_tiles((int)d->M, (int)d->N, d->format, &blocks);
      if (blocks < 0) return SZO_EUNSUPPORTED;
      T += blocks;
    }
    if (2 * T <= kNoAllocMaxPartials || !few_all) break;
  }
  // ... or, where the tiled kernel would run, the one-dense-pass kernel under szo_zo_step's conditions, if its partials fit.
  // (Not in place of the few-token path, but for layers beyond 128 tokens that only its split kernel takes: launched layer by
  // layer it does not fill the chip; one OPT block at 405 tokens 465 us with the few-token kernels, 479 with this one.)
  int64_t one_T = onepass_partials(descs, n, few_token_enabled() && small_m_eligible(descs, n, false, true, 2), false, false, true);
  if (2 * one_T > kNoAllocMaxPartials) one_T = 0;
  if (one_T) T = one_T;
  if (2 * T > kNoAllocMaxPartials) return SZO_EUNSUPPORTED;
  double* part = nullptr;
  int rc = noalloc_partials(&part);
  if (rc != SZO_OK) return rc;
  int64_t off = 0;
  for (int i = 0; i < n; ++i) {
    const szo_linear_desc* d = &descs[i];
    if (d->M == 0 || d->N == 0) continue;
    if (one_T) {
      rc = onepass_one(d, seed, step, eps, part + off, part + T + off, s);
      off += onepass_tiles(d);
    } else if (few_all) {
      rc = small_m_launch_one(d, seed, step, eps, 0, true, true, part + off, part + T + off, less, s);
      off += small_m_launch_partials(d, less);
    } else {
      const double scale = 1.0 / ((double)d->M * (double)d->N);
      int blocks;
      plan_tiles((int)d->M, (int)d->N, d->format, &blocks);
      rc = run_forward(d, seed, step, +1, eps, part + off, scale, s, false);
      if (rc == SZO_OK) rc = run_forward(d, seed, step, -1, eps, part + T + off, scale, s, true);
      off += blocks;
    }
    if (rc != SZO_OK) return rc;
  }
  if (T == 0) {                     // no layer with tokens: zero losses, g = 0
    rc = reduce_step(part, 0, eps, scalars, s);
    if (rc != SZO_OK) return rc;
  }
  return update_all(descs, n, seed, step, eps, lr, scalars, part, T, nullptr, s);
}

int szo_set_tile_config(int config) {
  if (config < 0 || config > 12) return SZO_EINVAL;
  g_tile_config = config;
  small_m_force_rblocks(config == 4 ? 2 : config == 5 ? 3 : 0);
  small_m_force_stream_once(config == 7 || config == 10);
  small_m_force_split(config == 8 ? 1 : config == 9 || config == 10 ? -1 : 0);
  onepass_force(config == 11 ? 1 : config == 0 ? 0 : -1);
  return SZO_OK;
}

int szo_linear_fwd(const szo_linear_desc* desc, uint64_t seed, uint64_t step, int sign, float eps, void* stream) {
  const int rc = validate_desc(desc, sign, true, false);
  if (rc != SZO_OK) return rc;
  if (desc->M == 0 || desc->N == 0) return SZO_OK;
  if (few_token_enabled() && small_m_takes_forward(desc, sign != 0 && eps != 0.0f))
    return small_m_launch_one(desc, seed, step, sign == 0 ? 0.0f : eps, sign == 0 ? 1 : sign, false, false, nullptr, nullptr,
                              kBandsInParts, (hipStream_t)stream);
  return run_forward(desc, seed, step, sign, eps, nullptr, 0.0, (hipStream_t)stream);
}

int szo_linear_fwd_mse(const szo_linear_desc* desc, uint64_t seed, uint64_t step, int sign, float eps,
                       double scale, double* loss_acc, void* workspace, void* stream) {
  int rc = validate_desc(desc, sign, false, true);
  if (rc != SZO_OK) return rc;
  if (!loss_acc || !workspace || ((uintptr_t)workspace & 7)) return SZO_EINVAL;
  if (desc->M == 0 || desc->N == 0) return SZO_OK;
  // the few-token kernels compute both signs at once: make the requested one the "+" forward.  Their scale is that of a
  // step's loss, and both signs' partials have to fit.
  const bool few = few_token_enabled() && small_m_takes_forward(desc, sign != 0 && eps != 0.0f) && scale == 1.0 / ((double)desc->M * (double)desc->N);
  const int64_t nb = few ? small_m_launch_partials(desc, kBandsInParts) : 0;
  if (few && 2 * nb <= kMaxLossPartials) {
    rc = small_m_launch_one(desc, seed, step, (float)sign * eps, desc->y ? 1 : 0, true, false, partial_area(workspace),
                            partial_area(workspace) + nb, kBandsInParts, (hipStream_t)stream);
    if (rc != SZO_OK) return rc;
    return reduce_partials(partial_area(workspace), (int)nb, 1.0, loss_acc, (hipStream_t)stream);
  }
  int blocks;
  plan_tiles((int)desc->M, (int)desc->N, desc->format, &blocks);
  if (blocks < 0 || blocks > kMaxLossPartials) return SZO_EUNSUPPORTED;
  rc = run_forward(desc, seed, step, sign, eps, partial_area(workspace), scale, (hipStream_t)stream);
  if (rc != SZO_OK) return rc;
  return reduce_partials(partial_area(workspace), blocks, 1.0, loss_acc, (hipStream_t)stream);
}

size_t szo_step_workspace_bytes(const szo_linear_desc* descs, int n, int flags) {
  if (n <= 0) return kSmallWorkspaceBytes;
  if (!descs) return kWorkspaceBytes;
  for (int i = 0; i < n; ++i)                               // copies are counted by their x: only of a step that would run
    if (validate_desc(&descs[i], 1, !(flags & SZO_STEP_FUSED_LOSS), true) != SZO_OK) return kWorkspaceBytes;
  const StepRoute route = step_route(descs, n, flags);
  static thread_local SharedPlan plan;
  if (!(route.instead_of_onepass || route.instead_of_two) || !plan.make(descs, n)) return kSmallWorkspaceBytes;
  return kWorkspaceBytes - kCopyAreaBytes + plan.bytes;
}

int szo_zo_step(const szo_linear_desc* descs, int n, uint64_t seed, uint64_t step, float eps, float lr,
                double* scalars, void* workspace, int flags, void* stream) {
  if (n < 0 || (n > 0 && !descs) || !scalars || !workspace || ((uintptr_t)workspace & 7)) return SZO_EINVAL;
  hipStream_t s = (hipStream_t)stream;
  // The step's descriptor tables travel through pinned host buffers that later calls reuse: a captured
  // step would replay stale tables.
  if (stream_is_capturing(s)) return SZO_EUNSUPPORTED;
  const bool fuse = flags & SZO_STEP_FUSED_LOSS;
  int64_t total = 0;                // workgroups = loss partials of one pass
  for (int i = 0; i < n; ++i) {     // reject everything before anything is enqueued
    const int rc = validate_desc(&descs[i], 1, !fuse, true);
    if (rc != SZO_OK) return rc;
    // the update touches every layer's values, also those of a layer without tokens
    if (descs[i].nnz > 0 && (!descs[i].sp_val || ((uintptr_t)descs[i].sp_val & 15))) return SZO_EINVAL;
    if (descs[i].M == 0 || descs[i].N == 0) continue;
    int blocks;
    plan_tiles((int)descs[i].M, (int)descs[i].N, descs[i].format, &blocks);
    if (blocks < 0) return SZO_EUNSUPPORTED;
    total += blocks;
  }
  int rc;
  void* const table_dev = (char*)workspace + kWorkspaceTableOffset;
  const StepRoute route = step_route(descs, n, flags);
  // Many tokens, one set of activations: the dense product once for both forwards (szo_onepass.hip; in large launches with rounded weights
  // the tiled kernel).
  {
    int64_t T = 0;
    rc = route.instead_of_onepass ? shared_forwards(descs, n, true, seed, step, eps, table_dev, copy_area(workspace), partial_area(workspace), &T, s) : SZO_EUNSUPPORTED;
    if (rc == SZO_EUNSUPPORTED)
      rc = onepass_forwards(descs, n, seed, step, eps, route.few_rule, route.asked_for, !fuse, table_dev, partial_area(workspace), &T, s);
    if (rc == SZO_OK) return update_all(descs, n, seed, step, eps, lr, scalars, partial_area(workspace), T, table_dev, s);
    if (rc != SZO_EUNSUPPORTED) return rc;      // otherwise nothing was enqueued
  }
  if (route.few) {
    rc = small_m_step(descs, n, seed, step, eps, lr, table_dev, partial_area(workspace), 0, scalars, true, s);
    if (rc != SZO_EUNSUPPORTED) return rc;      // too many slices for the table: nothing was enqueued, take the tiled path
  }
  if (fuse) {
    int64_t T = 0;
    rc = route.instead_of_two ? shared_forwards(descs, n, false, seed, step, eps, table_dev, copy_area(workspace), partial_area(workspace), &T, s) : SZO_EUNSUPPORTED;
    if (rc == SZO_EUNSUPPORTED) rc = grouped_forwards(descs, n, seed, step, eps, table_dev, partial_area(workspace), &T, s);
    if (rc == SZO_OK)
      return update_all(descs, n, seed, step, eps, lr, scalars, partial_area(workspace), T, table_dev, s);
    if (rc != SZO_EUNSUPPORTED) return rc;
  }
  if (fuse && 2 * total > kMaxLossPartials) return SZO_EUNSUPPORTED;
  if (!fuse) {
    rc = zero_words(scalars, 6, s);
    if (rc != SZO_OK) return rc;
  }
  for (int pass = 0; pass < 2; ++pass) {
    const int sign = pass == 0 ? +1 : -1;
    double* part = partial_area(workspace) + (size_t)pass * (size_t)total;
    for (int i = 0; i < n; ++i) {
      const szo_linear_desc* d = &descs[i];
      if (d->M == 0 || d->N == 0) continue;
      const double scale = 1.0 / ((double)d->M * (double)d->N);
      if (fuse) {
        int blocks;
        plan_tiles((int)d->M, (int)d->N, d->format, &blocks);
        rc = run_forward(d, seed, step, sign, eps, part, scale, s, pass == 1);
        part += blocks;
      } else {
        rc = run_forward(d, seed, step, sign, eps, nullptr, 0.0, s, pass == 1);
        if (rc == SZO_OK) rc = szo_mse_loss(d->y, d->target, d->M * d->N, scale, scalars + pass, workspace, s);
      }
      if (rc != SZO_OK) return rc;
    }
  }
  if (!fuse || total == 0) {        // no layer with tokens: zero losses, g = 0
    rc = fuse ? reduce_step(partial_area(workspace), 0, eps, scalars, s) : szo_spsa_g(scalars, scalars + 1, eps, scalars + 2, s);
    if (rc != SZO_OK) return rc;
  }
  return update_all(descs, n, seed, step, eps, lr, scalars, partial_area(workspace), fuse ? total : 0, table_dev, s);
}

}  // extern "C"
