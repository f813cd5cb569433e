// Grouped dequantize-GEMM, tile kernel for large buckets (prefill, images).
//
// Each sample is processed by its selected expert only (MoQE Section 3.1); when an expert's bucket
// holds hundreds of rows the work is a dense contraction and belongs on the matrix cores.  A
// work-group of 4 waves owns 128 or 64 bucket rows x 256 weight rows of one expert, or 64 x 128 (for the SiLU-gated
// pair: half of them gate rows and half the up rows of the same features, so the gate meets its up value in
// registers); a wave owns all the rows x a quarter of the weight rows.  Two work-groups share a CU (256 registers per
// wave), three of the narrow ones, and meet at their barriers independently, so one computes while the others wait.
//
// What bounds it is issue: a SIMD spends about 8 cycles issuing a matrix operation (the matrix pipe needs 16 for 16x16x32, 32 for 32x32x16)
// and 4 per vector instruction among them, so two of those per 16x16x32 operation are free, four to six per 32x32x16 one (probes with
// two waves on a SIMD: 64 among 512 clocks of matrix operations take 583 and 540, 128 take 848 and 678).  Hence:
//  * 128 rows per wave: a packed tile is unpacked once for eight matrix operations per operand (once for four
//    with 64 rows).
//  * Activations go from memory to LDS directly (buffer loads with the LDS as destination, 16 bytes per lane),
//    gathered through the permutation: no registers but, in the small tile, their offsets, and no vector instructions.  Rows of 256 bytes (128 for
//    int8 rows), 16-byte units XOR-swizzled by the row - the lane that fills a unit loads the swizzled column -
//    so that the 16-byte-per-lane operand reads are free of bank conflicts; double-buffered, one barrier per k-step.
//  * Weights never touch LDS: the packed layout already is the matrix-core operand order, so each
//    wave loads the four packed 16-row tiles of its 64 weight rows with one coalesced 16-byte-per-
//    lane load each (two k-steps ahead) and unpacks them in registers to exact bf16 operands BASE + c/2.
//  * Offset and zero-point are removed with the row sums of the activations.  Each wave sums a quarter of the
//    rows (an MFMA against ones) and hands the sums to the others through LDS, where they are read after the
//    k-step's barrier: a group of 128 leaves at the head of the next k-step.  (Groups of 64 take the small tile,
//    whose registers hold the wave's own sums.)  Per-channel formats subtract off * (row sum over all of k) at the end.
//    Removing the terms of several groups at once, as one matrix operation, is cheaper, but the uncorrected
//    sums grow and fp32 loses 3 (activations of mean 0) to 20 times (mean 0.5) as much: not done.
//  * Steps with many vector instructions (groups of 128; int8 and int6 on 64 x 256) use 32x32x16 operations, the next operand's unpacking between them.
//  * Per-group scales use ONE accumulator: entering group g the accumulator is multiplied by s_{g-1}/s_g, so
//    that it always holds the sum in units of the current group's scale, and the last scale multiplies the
//    result.  No weight is rounded; the extra roundings are one fp32 multiply per group on the accumulator.
//
// Measured on 8192 rows, k 11008, n 4096 of one format, launches back to back for 0.2 s, and before the 32 x 32 products, the priorities and the
// scales in registers: int4 per channel 1415 TFLOP/s (1407), int4 g128 1265 (1142), int3 g128 1189 (1072), int8 1323 (1324), int6 1089 (1036, small tile),
// groups of 64 850 (833, small tile), W8A8 2555 (2548); a library bf16 product of this size reaches 1586 (for 0.4 s, where int4 per channel reaches 1360).  With all-zero
// activations, the same instructions, that is 1722: long launches are held by power.
#include "qgemm_device.h"

#include <algorithm>
#include <cmath>
#include <cstring>

namespace moqe {

constexpr int TWAVES = 4;                // all along the weight rows
constexpr int TBM_MAX = 128;             // bucket rows of the large tile (8 blocks of 16); the others have 64

// What the launcher works out on the host for one launch.
struct TileGeom {
  uint64_t order_bits;                // 4 bits per position: experts in the order their row tiles are enumerated, dearest format first
  uint32_t a_bytes;                   // bytes of the activation matrix (16-bit rows)
  // one word, which the kernel reads at its head
  uint8_t  patch_n_log2;              // a patch is 2^patch_n_log2 weight tiles x PATCH_M row tiles
  uint8_t  tbm;                       // bucket rows per tile, 128 or 64
  uint8_t  products_first;            // 32 x 32 x 16 products of a wave go ahead of the other waves' instructions
};

struct TileLds {
  uint8_t* buf[2];                    // staged activations, one k-step each
  float*   xs;                        // [2][TBM_MAX] row sums of the last two k-steps (per-channel formats: over all of k)
  int32_t* drow;                      // [TBM_MAX] destination row of each tile row, -1: none
  float*   sx;                        // [TBM_MAX] scale of each int8 activation row
  uint32_t* src;                      // [TBM_MAX] byte offset of each tile row's source (convolution: of its pixel)
  uint16_t* taps;                     // [TBM_MAX] convolution: bit t set = filter tap t of the row's pixel lies inside its image
};

// s_waitcnt: at most `vm` vector-memory requests in flight, all LDS traffic done
template <int VM> static __device__ __forceinline__ void wait_vm_lds() {
  static_assert(VM < 64, "6-bit counter");
  __builtin_amdgcn_s_waitcnt((VM & 15) | (7 << 4) | (0 << 8) | ((VM >> 4) << 14));
}
static __device__ __forceinline__ void group_barrier() {
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
  __builtin_amdgcn_sched_barrier(0);
}

// The lane's number, worked out where it is asked for.  As an expression of threadIdx it is one value for the whole kernel, which the 128-row tiles of groups of 128, whose
// k-loop fills all registers, kept in scratch memory: every format then read it back ahead of its first requests and of its results (plain launches of
// 64 x 256 tiles, k 1152, 1/2 to 3.5 rounds: W8A8 1.03 - 1.06 times as long, int4 in groups of 64 1.09 - 1.14).
static __device__ __forceinline__ int lane_here() {
  int lane;
  asm volatile("v_mbcnt_lo_u32_b32 %0, -1, 0\n\tv_mbcnt_hi_u32_b32 %0, -1, %0" : "=v"(lane));
  __builtin_assume(lane >= 0 && lane < 64);
  return lane;
}

// Priority 1 for the wave, always or if `on` (uniform).  The branch is inside the asm: as control flow of the program it splits the k-step, and 19 registers are
// spilled in the loop.  Groups of 64, which would meet it twice a k-step (a linear block of 32 x 16 rows of 256 14.85 -> 15.0 us), and the convolution have none.
template <bool ALWAYS> static __device__ __forceinline__ void raise_priority([[maybe_unused]] int on) {
  if constexpr (!ALWAYS) __builtin_amdgcn_sched_barrier(0);          // s_setprio itself is one
  if constexpr (ALWAYS) __builtin_amdgcn_s_setprio(1);
  else asm volatile("s_cmp_lg_u32 %0, 0\n\ts_cbranch_scc0 .Lkeep_priority%=\n\ts_setprio 1\n.Lkeep_priority%=:" : : "s"(on) : "scc");
}

typedef float f32x16 __attribute__((ext_vector_type(16)));
static __device__ __forceinline__ f32x16 mfma_bf16_32(const u32x4& a, const bf16x8& b, f32x16 c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a), b, c, 0, 0, 0);
}

template <int I, int N, typename F> static __device__ __forceinline__ void unroll(F&& f) {
  if constexpr (I < N) {
    f(std::integral_constant<int, I>{});
    unroll<I + 1, N>(f);
  }
}
// The order of a unit of the k-step: LDS reads first, then N products with vector instructions between them.
template <int N> static __device__ __forceinline__ void interleave() {
  __builtin_amdgcn_sched_group_barrier(0x100, 2, 0);
#pragma unroll
  for (int i = 0; i < N; ++i) {
    __builtin_amdgcn_sched_group_barrier(0x8, 1, 0);
    __builtin_amdgcn_sched_group_barrier(0x2, 6, 0);
  }
}

typedef __attribute__((address_space(3))) void lds_void;
typedef const __attribute__((address_space(1))) uint8_t* glb_bytes;

template <int TMB, int TNB, int FMT, int GM, bool GATEUP, bool CONV>
static __device__ __forceinline__ void tile_task(const GemmArgs& ga, const TileGeom& tg, const ExpertDev& ex, const int off_e, const int M_e,
                                                 const int m0, const int ntile, const int own_wave, const TileLds& sh) {
  constexpr bool A8 = (FMT == FMT_I8A8);
  constexpr int NR = Raw<FMT>::N;
  constexpr int GPT = GM == GM_PC ? 0 : (GM == GM_G128 ? 1 : 2);
  constexpr int EB = A8 ? 1 : 2;
  constexpr int TBM = TMB * 16;
  constexpr int HB = GATEUP ? TNB / 2 : TNB;         // weight blocks of the first matrix; the others are the second one's (up)
  constexpr int OWN = TMB / TWAVES;                  // row blocks whose sums this wave takes
  // Products of 32 x 32 x 16 instead of 16 x 16 x 32: half as many to issue, and four to six vector instructions in the shadow of each.  Taken where a step holds
  // many of those: groups of 128, and the longer unpacking of int8 and int6 codes on 64 x 256 (8192 rows, k 11008, n 4096: int6 729 -> 690 us; 2048 rows, k and n 4096: int8
  // 71.4 -> 65.2, int6 74 -> 71.5).  On 64 x 128 they cost those codes 1 to 8 % in launches of a round and more, and gated int6 ones 1.03 to 1.5 times the time (the scales of a
  // block of 16 gate and 16 up rows came through scratch memory).  Not for int4 per channel (2048 rows 61.9 -> 62.5), not for the convolution (256 images 80 -> 85): power,
  // and less to hide.
  constexpr bool M32 = GM == GM_G128 || (GM == GM_PC && TMB == 4 && TNB == 4 && !CONV && (FMT == FMT_I8 || FMT == FMT_N6));
  // What a lane holds of the results: NQ quads of neighbouring rows x NC weight rows.
  constexpr int NQ = M32 ? 2 * TMB : TMB, NC = M32 ? TNB / 2 : TNB;
  constexpr bool MIXED = M32 && GATEUP && TNB == 2;  // a block of 32 weight rows is 16 gate rows and the 16 up rows of the same features
  constexpr int AROW = 128 * EB;                     // LDS bytes of a staged row
  constexpr int BLK = 16 * AROW;                     // ... of a block of 16 rows
  constexpr int A_UNITS = AROW / 16;                 // 16-byte units per row
  constexpr int A_IT_ROWS = TWAVES * 64 / A_UNITS;   // rows the work-group stages per request
  constexpr int A_ITERS = TBM / A_IT_ROWS;
  // The large tile's registers hold one k-step of 8-bit codes, refilled by halves as they are used up; smaller codes, and the small
  // tile, keep two k-steps.
  // Two row blocks' operands are read from LDS while the two before are multiplied, and the wave's row sums are taken along the way.
  constexpr bool HALVES = TMB == 8 && FMT == FMT_I8;
  constexpr int W_LOADS = TNB * (FMT == FMT_N4 ? 1 : 2) + (GPT ? 2 : 0);   // weight requests of a k-step
  constexpr float BASE = CodeMap<FMT>::BASE, CM = CodeMap<FMT>::CM, INV_CM = 1.f / CodeMap<FMT>::CM;

  constexpr bool FULL = TNB == 4 && !CONV;           // the kernels whose registers are all taken
  const int tid = FULL ? 0 : int(threadIdx.x);
  const int wave = FULL ? own_wave : __builtin_amdgcn_readfirstlane(tid >> 6);       // uniform: keeps tile addresses scalar
  int lane = FULL ? lane_here() : tid & 63, lr = lane & 15, lq = lane >> 4;
  const int KT = ga.k >> 7, NT = ga.n >> 4;
  const int T = ga.T;
  const float off_sym = BASE + CM * float(ex.zc);
  const FragK<FMT> fk = frag_constants<FMT>();

  // ---- the four packed weight tiles of this wave (16 weight rows each) -----------------------------
  const uint8_t* blob[TNB];
  uint32_t tbase[TNB];                        // index of the tile's first k-step inside the blob
#pragma unroll
  for (int b = 0; b < TNB; ++b) {
    const int nt16 = (ntile * TWAVES + wave) * HB + b % HB;       // gate/up: gate rows, then the up rows of the same features
    blob[b] = ex.w[b / HB];
    tbase[b] = uint32_t((nt16 < NT ? nt16 : 0) * KT);   // clamped: rows outside the matrix are computed on other rows' codes, never stored
  }
  // The weight rows of this lane's results: tile c, or of tiles 2c and 2c + 1 the one of the lane's half of its block's 32 columns.
  auto tile_of = [&](int c) { return M32 ? 2 * c + (lq & 1) : c; };
  auto ncol = [&](int c) { return ((ntile * TWAVES + wave) * HB + tile_of(c) % HB) * 16 + lr; };      // weight row (plain) / feature (gate-up)

  // ---- weight ring: two k-steps in flight ------------------------------------------------------------
  // All of it waits in registers.  Of scales and zero-points a lane holds those of one weight row (lane l: row l % 16 of block l / 16; zero-points as the
  // aligned dword that holds them); what it makes of them is handed round when a group is entered (spread()).  They are plain loads: as transfers to LDS
  // (global_load_lds) they count as loads that may touch LDS, and as long as one is on its way the compiler lets every wait for an LDS operand be
  // a wait for all of them: no operand could be asked for ahead (groups of 64, 8192 rows, k 11008, n 4096: 894 -> 872 us; 512 rows, k and n 4096: 54.2 -> 52.7).
  const buf_rsrc w_rsrc[2] = {blob_rsrc(ex.w[0]), blob_rsrc(ex.w[GATEUP ? 1 : 0])};
  uint32_t raw[HALVES ? 1 : 2][TNB][NR];
  glb_bytes sc_src = nullptr, zp_src = nullptr;
  uint32_t szr[2][3];                                  // scales of a k-step's groups, zero-points
  if constexpr (GPT > 0) {
    uint32_t t = tbase[0];
    const uint8_t* bl = blob[0];
#pragma unroll
    for (int b = 1; b < TNB; ++b) {
      t = lq % TNB == b ? tbase[b] : t;
      bl = lq % TNB == b ? blob[b] : bl;
    }
    sc_src = glb_bytes(bl) + (ex.scale_off + t * uint32_t(64 * GPT) + uint32_t(lr * 4 * GPT));
    zp_src = glb_bytes(bl) + (ex.zero_off + t * uint32_t(16 * GPT) + uint32_t((lr * GPT) & ~3));
  }
  auto issue_w = [&](int p, int kt_want) {
    const uint32_t kt = uint32_t(min(kt_want, KT - 1));
#pragma unroll
    for (int b = 0; b < TNB; ++b) load_raw<FMT>(raw[p][b], w_rsrc[b / HB], (tbase[b] + kt) * ex.tile_bytes, lane);
    if constexpr (GPT > 0) {
      if constexpr (GPT == 1) {
        szr[p][0] = *reinterpret_cast<const __attribute__((address_space(1))) uint32_t*>(sc_src + kt * 64u);
      } else {
        const u32x2 v = *reinterpret_cast<const __attribute__((address_space(1))) u32x2*>(sc_src + kt * 128u);
        szr[p][0] = v.x; szr[p][1] = v.y;
      }
      szr[p][2] = *reinterpret_cast<const __attribute__((address_space(1))) uint32_t*>(zp_src + kt * uint32_t(16 * GPT));
    }
  };
  [[maybe_unused]] auto issue_half = [&](int h, int kt_want) {          // 8-bit codes of steps 2h and 2h + 1 of a k-step
    const uint32_t kt = uint32_t(min(kt_want, KT - 1));
#pragma unroll
    for (int b = 0; b < TNB; ++b) {
      const buf_rsrc rs = w_rsrc[b / HB];
      const uint32_t at = (tbase[b] + kt) * ex.tile_bytes;
      const u32x4 v = buf_load128(rs, lane * 16 + h * 1024, at);
      raw[0][b][4 * h] = v.x; raw[0][b][4 * h + 1] = v.y; raw[0][b][4 * h + 2] = v.z; raw[0][b][4 * h + 3] = v.w;
    }
  };
  const uint32_t zp_shift = GPT == 2 ? 16u * (uint32_t(lr) & 1u) : 8u * (uint32_t(lr) & 3u);

  // ---- activation rows this lane copies per k-step ------------------------------------------------
  // Request i of a wave fills 1 KiB of LDS, lane after lane: rows i * A_IT_ROWS + wave * (64 / A_UNITS) + lane / A_UNITS.  The
  // lane's unit of the row is the swizzled one, the same for every i (the swizzle looks at the row within its block of 16).
  const buf_rsrc a_rsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(A8 ? static_cast<const void*>(ga.a_q) : ga.a), 0,
                                                            A8 ? tg.a_bytes >> 1 : tg.a_bytes, 0x00020000);
  const int a_row0 = wave * (64 / A_UNITS) + lane / A_UNITS;
  const uint32_t a_col = uint32_t((lane % A_UNITS) ^ (A8 ? (a_row0 >> 1) & 7 : a_row0 & 15)) * 16u;
  // Source and destination of the tile's rows and, for int8 activations, their scale: looked up once, one row per thread, and kept in LDS,
  // because registers are what this kernel is short of.  Rows past the bucket repeat its last row; destination -1.
  // The small tile keeps the offsets of the rows that a lane copies (2 to 4) in registers: each wave looks its own 16 rows up, ahead of
  // the weights (loads come back in order), and its lanes hand the offsets round.  Through the table the first request would wait for a
  // barrier, and with it for the first weights, and the requests of every k-step for LDS.  (Groups of 64 and 6-bit codes, with the
  // longest k-steps and the fewest registers to spare, are 2 % faster with the table.)
  constexpr bool DIRECT = TMB == 4 && !CONV && GM != GM_G64 && FMT != FMT_N6;
  constexpr int RPW = 64 / A_UNITS;          // rows a wave copies per request
  static_assert(!DIRECT || A_ITERS * RPW == 16, "a wave copies 16 rows of the small tile");
  const int t_row = DIRECT ? ((lane & 15) / RPW) * A_IT_ROWS + wave * RPW + (lane & 15) % RPW : FULL ? wave * 64 + lane : tid;
  const bool t_mine = DIRECT ? lane < 16 : t_row < TBM;
  int t_src = 0, t_dst = 0, t_rin = 0;
  float t_sx = 0.f;
  auto look_up = [&]() {
    const int m = min(m0 + t_row, M_e - 1);
    const bool one_row = T == 1;             // uniform: the division is some forty instructions
    const int smp = off_e + (one_row ? m : m / T);
    t_rin = one_row ? 0 : m - (smp - off_e) * T;
    t_src = t_dst = smp;                     // the sample, for now
    if constexpr (!A8) {
      if (ga.a_perm != nullptr) t_src = ga.a_perm[smp];       // int8 rows are in bucket order
    }
    if constexpr (A8) t_sx = ga.a_scale[smp * T + t_rin];
    if constexpr (!GATEUP) {
      if (ga.y_perm) t_dst = ga.y_perm[smp];
    }
  };
  // each matrix is smaller than 4 GiB: 32-bit byte offsets
  auto row_bytes = [&]() { return uint32_t(t_src * T + t_rin) * uint32_t(CONV ? ga.conv_c : ga.k) * uint32_t(EB); };
  auto fill_rows = [&]() {
    if (!t_mine) return;
    if constexpr (!DIRECT) sh.src[t_row] = row_bytes();
    if constexpr (CONV) {
      const int py = t_rin / ga.conv_w, px = t_rin - py * ga.conv_w;    // the pixel inside its image
      uint32_t taps = 0;
#pragma unroll
      for (int t = 0; t < 9; ++t) {
        const int yy = py + t / 3 - 1, xx = px + t % 3 - 1;
        if (yy >= 0 && yy < ga.conv_h && xx >= 0 && xx < ga.conv_w) taps |= 1u << t;
      }
      sh.taps[t_row] = uint16_t(taps);
    }
    if constexpr (A8) sh.sx[t_row] = t_sx;
    sh.drow[t_row] = m0 + t_row < M_e ? t_dst * T + t_rin : -1;
    sh.xs[TBM_MAX + t_row] = 0.f;            // what the first k-step takes for the sums before it
  };
  uint32_t a_off[DIRECT ? A_ITERS : 1];
  if constexpr (DIRECT) look_up();
  __builtin_amdgcn_sched_barrier(0);
  if constexpr (!HALVES) issue_w(0, 0);      // the first step's weights
  __builtin_amdgcn_sched_barrier(0);
  if constexpr (DIRECT) {
    const uint32_t mine = row_bytes();
#pragma unroll
    for (int i = 0; i < A_ITERS; ++i) a_off[i] = uint32_t(__shfl(int(mine), i * RPW + lane / A_UNITS)) + a_col;
  } else {
    if (t_mine) look_up();
    fill_rows();
    __syncthreads();
  }
  // Convolution: conv_c is a multiple of 128 (9 conv_c is), so a k-step lies inside ONE filter tap (k = tap * C + channel): the
  // lane's unit is 16 contiguous bytes of the pixel at that tap's offset.  Outside the image the offset is past the matrix, which
  // reads as zeros (the matrix ends on a multiple of 256 bytes below 4 GiB).
  // The offsets of a k-step are worked out at the end of the step before (a_prepare), so that its requests can leave right behind the barrier.
  constexpr bool EARLY = GM != GM_PC || CONV;
  uint32_t a_now[DIRECT ? 1 : A_ITERS];
  int tap = 0, tap_ch = 0;                           // convolution: filter tap and first channel of the step that a_prepare() looks at next
  auto a_prepare = [&]() {
    if constexpr (!DIRECT) {
      int delta = 0;
      if constexpr (CONV) {
        const int ty = tap / 3;
        delta = (((ty - 1) * ga.conv_w + (tap - ty * 3 - 1)) * ga.conv_c + tap_ch) * 2;
      }
#pragma unroll
      for (int i = 0; i < A_ITERS; ++i) {
        uint32_t off = sh.src[i * A_IT_ROWS + a_row0] + a_col;
        if constexpr (CONV) off = ((uint32_t(sh.taps[i * A_IT_ROWS + a_row0]) >> tap) & 1u) ? off + uint32_t(delta) : 0xFFFFFF00u;
        a_now[i] = off;
      }
      if constexpr (CONV) {
        tap_ch += 128;
        if (tap_ch == ga.conv_c) { tap_ch = 0; ++tap; }      // behind the last step there is no tap: nothing is read
      }
    }
  };
  auto a_fetch = [&](int kt_want, uint8_t* buf) {
    if constexpr (!EARLY) a_prepare();
    const uint32_t koff = CONV ? 0u : uint32_t(min(kt_want, KT - 1)) * uint32_t(AROW);
#pragma unroll
    for (int i = 0; i < A_ITERS; ++i)
      __builtin_amdgcn_raw_ptr_buffer_load_lds(a_rsrc, (lds_void*)(buf + (i * TWAVES + wave) * 1024), 16, int(DIRECT ? a_off[DIRECT ? i : 0] : a_now[DIRECT ? 0 : i]),
                                               int(koff), 0, 0);
  };

  // Register row block rb of this wave is the tile's row block rb ^ rot: block 0 holds the rows whose sums the wave takes.
  const int rot = M32 ? wave * OWN / 2 : wave * OWN;
  f32x4 tot[M32 ? 1 : TMB][TNB];                   // 16 x 16: fp32 sums in units of the current group's scale; int8 path: int32 bit patterns
  f32x16 tot32[M32 ? TMB / 2 : 1][M32 ? NC : 1];   // 32 x 32: the same
  f32x4 xs_own[OWN];          // row sums of the wave's own blocks of 16 over the k-step (per-channel formats: over all of k)
  // Of the lane's own weight row (as in szr): scale of the group that the accumulators are expressed in; groups of 128: offset + zero-point of the
  // group whose row sums are still to be removed.
  float s_cur = 1.f, o_last = 0.f;
  const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int mb = 0; mb < (M32 ? 1 : TMB); ++mb)
#pragma unroll
    for (int b = 0; b < TNB; ++b) tot[mb][b] = zero;
#pragma unroll
  for (int rb = 0; rb < (M32 ? TMB / 2 : 1); ++rb)
#pragma unroll
    for (int c = 0; c < (M32 ? NC : 1); ++c)
#pragma unroll
      for (int r = 0; r < 16; ++r) tot32[rb][c][r] = 0.f;
#pragma unroll
  for (int i = 0; i < OWN; ++i) xs_own[i] = zero;
  const u32x4 ones = {0x3F803F80u, 0x3F803F80u, 0x3F803F80u, 0x3F803F80u};
  const uint32_t half_ones = ((lq ^ lr) & 1) == 0 ? 0x3F803F80u : 0u;
  const u32x4 own_mask = {half_ones, half_ones, half_ones, half_ones};
  // Tile row of register 0 of quad q, and what the quad holds
  auto quad_row = [&](int q) { return M32 ? ((q >> 2) ^ rot) * 32 + (q & 3) * 8 + (lane >> 5) * 4 : (q ^ rot) * 16 + lq * 4; };
  auto res = [&](int q, int c, int r) -> float { if constexpr (M32) return tot32[q >> 2][c][(q & 3) * 4 + r]; else return tot[q][c][r]; };
  // A value of the lanes' own weight rows as the lanes need it for their results
  auto spread = [&](float v, float (&out)[NC]) {
    const uint32_t u = __float_as_uint(v);
    if constexpr (M32 && TNB == 2) {
      out[0] = v;                                      // lanes 32 .. 63 hold the same rows
    } else if constexpr (M32) {
      const auto h = __builtin_amdgcn_permlane32_swap(u, u, false, false);
      out[0] = __uint_as_float(h[0]); out[1] = __uint_as_float(h[1]);
    } else {
      uint32_t half[2] = {u, u};
      if constexpr (TNB == 4) {
        const auto h = __builtin_amdgcn_permlane32_swap(u, u, false, false);
        half[0] = h[0]; half[1] = h[1];
      }
#pragma unroll
      for (int b = 0; b < TNB; b += 2) {
        const auto r = __builtin_amdgcn_permlane16_swap(half[b / 2], half[b / 2], false, false);
        out[b] = __uint_as_float(r[0]); out[b + 1] = __uint_as_float(r[1]);
      }
    }
  };
  // Entering the group of scale s_new: what accumulators in units of s_cur are multiplied by: s_cur / s_new from the hardware reciprocal and one Newton
  // step (within an ulp or two of the true quotient; any error only moves rounding points, the factor is applied and divided out consistently).
  auto enter_group = [&](float s_new, float (&rho)[NC]) {
    float rinv = __builtin_amdgcn_rcpf(s_new);
    rinv = fmaf(fmaf(-s_new, rinv, 1.0f), rinv, rinv);
    spread(s_cur * rinv, rho);
    s_cur = __builtin_canonicalizef(s_new);          // an instruction, not a copy: copies end up behind the ring's next load, waiting for it
  };
  // operand reads: unit u = 4 j + lq of row lr of a block of 16; unit 4 j + 2 (lane / 32) + h of row lane % 32 of a block of 32
  const uint32_t a_lane = uint32_t(rot * BLK + lr * AROW + ((lq ^ (A8 ? (lr >> 1) & 7 : lr)) * 16));
  const uint32_t a_own = uint32_t(wave * OWN * BLK + lr * AROW + ((lq ^ lr) * 16));      // the wave's own rows, for their sums
  const uint32_t a_lane32 = uint32_t(rot * 2 * BLK + (lane & 31) * AROW + (((lane >> 5) * 2) ^ lr) * 16);

  // One k-step: activation operands from LDS buffer `abuf`, weights from ring slot p.
  auto compute = [&](int p, int kt, const uint8_t* abuf, auto fetch) {
    const int ps = HALVES ? 0 : p;
    // The ring values arrive through the loop's back edge; the fence keeps the optimizer from moving
    // arithmetic on them to the end of the previous iteration, right behind their loads.
    auto fence = [&](int first, int last) {
#pragma unroll
      for (int b = 0; b < TNB; ++b)
#pragma unroll
        for (int i = first; i < last; ++i) asm volatile("" : "+v"(raw[ps][b][i]));
      if constexpr (GPT > 0) {
#pragma unroll
        for (int i = 0; i < 3; ++i)
          if (i < GPT || i == 2) asm volatile("" : "+v"(szr[p][i]));
      }
    };
    if constexpr (!HALVES) fence(0, NR);
    else fence(0, 4);
    // unit u = 4 j + lq of block rb: the swizzle is an XOR, so block and step only flip bits of the lane's offset
    auto a_read = [&](int j, int rb) {
      const uint32_t o = (a_lane ^ uint32_t(j * 64) ^ uint32_t((rb & ~(OWN - 1)) * BLK)) + uint32_t((rb & (OWN - 1)) * BLK);
      return *reinterpret_cast<const u32x4*>(abuf + o);
    };
    auto a_read32 = [&](int j, int h, int rb) {
      return *reinterpret_cast<const u32x4*>(abuf + (a_lane32 ^ uint32_t(j * 64) ^ uint32_t(h * 16) ^ uint32_t(rb * 2 * BLK)));
    };
    if constexpr (A8) {
      fetch();
      __builtin_amdgcn_sched_barrier(0);
      // Pairs of row blocks; their operands are read PF pairs ahead (the small tile: all of them ahead of the first product).
      constexpr int PAIRS = TMB, PF = TMB == 4 ? PAIRS : 2, RING = TMB == 4 ? PAIRS : 3;
      u32x4 av[RING][2];
      auto a_pair = [&](int q) {
#pragma unroll
        for (int i = 0; i < 2; ++i) av[q % RING][i] = a_read(q / (TMB / 2), q % (TMB / 2) * 2 + i);
      };
#pragma unroll
      for (int q = 0; q < PF; ++q) a_pair(q);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int q = 0; q < PAIRS; ++q) {
        if (q + PF < PAIRS) a_pair(q + PF);
        if constexpr (TMB == 8) __builtin_amdgcn_sched_barrier(0);
        const int js = q / (TMB / 2);
#pragma unroll
        for (int i = 0; i < 2; ++i) {
          const int mb = q % (TMB / 2) * 2 + i;
#pragma unroll
          for (int b = 0; b < TNB; ++b) {
            const i32x4 bv = {int(raw[ps][b][js * 4 + 0]), int(raw[ps][b][js * 4 + 1]), int(raw[ps][b][js * 4 + 2]),
                              int(raw[ps][b][js * 4 + 3])};
            tot[mb][b] = __builtin_bit_cast(f32x4, __builtin_amdgcn_mfma_i32_16x16x64_i8(__builtin_bit_cast(i32x4, av[q % RING][i]), bv,
                                                                                         __builtin_bit_cast(i32x4, tot[mb][b]), 0, 0, 0));
          }
        }
        if constexpr (TMB == 8) __builtin_amdgcn_sched_barrier(0);
      }
    } else if constexpr (M32) {
      // A k-step is 8 (j, h) x RB / 2 units, each the products of two row blocks of 32 with the wave's NC blocks of weight rows.  Every unit asks for
      // the next one's activations and unpacks its share of the next (j, h)'s weights between its own products: four vector
      // instructions fit into the shadow of a 32 x 32 x 16 product, and none of them waits for LDS.
      constexpr int RB = TMB / 2, UNITS = 8 * (RB / 2), UPS = RB / 2;
      constexpr int PF = TMB == 8 ? 1 : 2;             // units that activations are asked for ahead: as many as registers allow
      u32x4 av[PF + 1][2];
      bf16x8 bv[2][NC];                                // weights of a (j, h) and of the next one
      auto a_unit = [&](int q) {
#pragma unroll
        for (int i = 0; i < 2; ++i) av[q % (PF + 1)][i] = a_read32(q / (2 * UPS), q / UPS % 2, q % UPS * 2 + i);
      };
      f32x4 x4[2][4];                                  // row sums of the previous k-step: of a row block and of the next one
      const float* src = sh.xs + (p ^ 1) * TBM_MAX;
      auto x_read = [&](int rb) {
#pragma unroll
        for (int i = 0; i < 4; ++i) x4[rb & 1][i] = *reinterpret_cast<const f32x4*>(src + quad_row(rb * 4 + i));
      };
      if constexpr (GM == GM_G128) x_read(0);
      __builtin_amdgcn_sched_barrier(0);
      u32x4 own[TMB == 4 ? 4 : 1];                     // the small tile's own rows, as operands of 16 rows, for their sums
      if constexpr (TMB == 4) {
#pragma unroll
        for (int j = 0; j < 4; ++j) own[j] = *reinterpret_cast<const u32x4*>(abuf + (a_own ^ uint32_t(j * 64)));
      }
#pragma unroll
      for (int q = 0; q < PF; ++q) a_unit(q);
      __builtin_amdgcn_sched_barrier(0);
      fetch();
      __builtin_amdgcn_sched_barrier(0);
      // The lanes of a loaded tile hold its 16 rows at four octets of columns; a 32 x 32 x 16 product wants 32 rows at two.  Swapping the odd rows of
      // 16 lanes of one tile with the even ones of the other gives the operands of octets 0 and 2, and of octets 1 and 3.
#pragma unroll
      for (int b = 0; b < TNB; b += 2)
#pragma unroll
        for (int i = 0; i < NR; ++i) {
          const auto v = __builtin_amdgcn_permlane16_swap(raw[p][b][i], raw[p][b + 1][i], false, false);
          raw[p][b][i] = v[0]; raw[p][b + 1][i] = v[1];
        }
#pragma unroll
      for (int c = 0; c < NC; ++c) bv[0][c] = frag<FMT, 0>(raw[p][2 * c], fk);
      if constexpr (GM == GM_G128) {
        float rho[NC], o[NC];
        spread(o_last, o);
        enter_group(__uint_as_float(szr[p][0]), rho);
        o_last = BASE + CM * float((szr[p][2] >> zp_shift) & 0xffu);
        // The previous k-step's group leaves here: its row sums have come from the waves that own the rows.
#pragma unroll
        for (int rb = 0; rb < RB; ++rb) {
          if (rb + 1 < RB) x_read(rb + 1);
          __builtin_amdgcn_sched_barrier(0);
#pragma unroll
          for (int c = 0; c < NC; ++c)
#pragma unroll
            for (int i = 0; i < 16; ++i) tot32[rb][c][i] = (tot32[rb][c][i] - o[c] * x4[rb & 1][i / 4][i % 4]) * rho[c];
          __builtin_amdgcn_sched_barrier(0);
        }
      }
      f32x4 sums = GM == GM_PC ? xs_own[0] : zero;
      // Products go ahead of the other work-groups' rescaling, so that one computes while another rescales: without it the work-groups of a CU fall into step
      // (8192 rows, k 11008, n 4096: int4 g128 630 -> 585 us, int3 653 -> 615; 2048 rows, k and n 4096: int4 77.8 -> 71.7, int3 85.7 -> 78.9).
      raise_priority<CONV || GM == GM_G64>(tg.products_first);
      unroll<0, UNITS>([&](auto qc) {
        constexpr int q = decltype(qc)::value, jh = q / UPS, pr = q % UPS;
        if constexpr (q + PF < UNITS) a_unit(q + PF);
        if constexpr (jh + 1 < 8) {                    // the next (j, h)'s weights
#pragma unroll
          for (int c = pr; c < NC; c += UPS) bv[(jh + 1) & 1][c] = frag<FMT, (jh + 1) / 2>(raw[p][2 * c + (jh + 1) % 2], fk);
        }
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
          for (int c = 0; c < NC; ++c) tot32[pr * 2 + i][c] = mfma_bf16_32(av[q % (PF + 1)][i], bv[jh & 1][c], tot32[pr * 2 + i][c]);
        // The wave's own row sums, with ones as the first operand.  Large tile: row block 0 as an operand of 16 rows is its rows 0 - 15 in the octets of
        // columns 0 and 2 and its rows 16 - 31 in the others, which ones in the even rows' even octets and the odd rows' odd ones keep apart where all are finite.
        if constexpr (TMB == 8 && pr == 0) sums = mfma_bf16(own_mask, __builtin_bit_cast(bf16x8, av[q % (PF + 1)][0]), sums);
        if constexpr (TMB == 4 && q < 4) sums = mfma_bf16(ones, __builtin_bit_cast(bf16x8, own[q]), sums);
        interleave<2 * NC>();
        __builtin_amdgcn_sched_barrier(0);
      });
      __builtin_amdgcn_s_setprio(0);
      if constexpr (TMB == 8) {
        // Zero times an infinity is NaN: a row that is not finite spoils the sum of the row 16 away from it.  So a wave whose sums are not all finite takes them
        // again by the same products, each row with the other's bits cleared: every finite row's sum is bit for bit the one it has among finite rows.  (Sums that
        // keep the rows apart for everyone, as dot products of a lane's own octets or as 4 x 4 x 4 products, made launches of 8192 rows 1 to 2 % longer.)
        if (__any(sums[0] * 0.f + sums[1] * 0.f != 0.f)) {
#pragma unroll
          for (int i = 0; i < 2; ++i) {
            f32x4 again = zero;
#pragma unroll 1
            for (int jh = 0; jh < 8; ++jh) {
              u32x4 v = a_read32(jh / 2, jh % 2, 0);
#pragma unroll
              for (int w = 0; w < 4; ++w) v[w] = (lq & 1) == i ? v[w] : 0u;
              again = mfma_bf16(own_mask, __builtin_bit_cast(bf16x8, v), again);
            }
            sums[i] = again[i];
          }
        }
      }
      if constexpr (GM == GM_PC) xs_own[0] = sums;
      if (GM == GM_G128 && lq == 0) {                  // for all waves
        sh.xs[p * TBM_MAX + wave * OWN * 16 + lr] = sums[0];
        if constexpr (OWN == 2) sh.xs[p * TBM_MAX + wave * OWN * 16 + 16 + lr] = sums[1];
      }
    } else {                                           // scales per channel, groups of 64
      u32x4 av[2][2];                                  // operands of two row blocks, read while the two before are multiplied
      if constexpr (!EARLY) { fetch(); __builtin_amdgcn_sched_barrier(0); }
#pragma unroll
      for (int i = 0; i < 2; ++i) av[0][i] = a_read(0, i);
      if constexpr (EARLY) { __builtin_amdgcn_sched_barrier(0); fetch(); __builtin_amdgcn_sched_barrier(0); }
      f32x4 xs[GM == GM_G64 ? TMB : 1];                // groups of 64: row sums of the current group, every wave its own
      auto do_j = [&](auto jc) {
        constexpr int J = decltype(jc)::value, G = J / 2;
        if constexpr (GM == GM_G64 && J % 2 == 0) {    // entering a group: accumulators into its scale's units
          float rho[NC];
          enter_group(__uint_as_float(szr[p][G]), rho);
#pragma unroll
          for (int b = 0; b < TNB; ++b)
#pragma unroll
            for (int mb = 0; mb < TMB; ++mb)
#pragma unroll
              for (int r = 0; r < 4; ++r) tot[mb][b][r] *= rho[b];
        }
        if constexpr (GM == GM_G64) {                  // as for 32 x 32 products
          __builtin_amdgcn_sched_barrier(0);
          raise_priority<CONV || GM == GM_G64>(tg.products_first);
        }
        bf16x8 bv[TNB];
#pragma unroll
        for (int b = 0; b < TNB; ++b) bv[b] = frag<FMT, J>(raw[ps][b], fk);
#pragma unroll
        for (int pr = 0; pr < TMB / 2; ++pr) {
          constexpr int last = 4 * (TMB / 2) - 1;
          const int q = J * (TMB / 2) + pr;
          if (q < last) {
#pragma unroll
            for (int i = 0; i < 2; ++i) av[(q + 1) & 1][i] = a_read((q + 1) / (TMB / 2), (q + 1) % (TMB / 2) * 2 + i);
          }
          __builtin_amdgcn_sched_barrier(0);
#pragma unroll
          for (int i = 0; i < 2; ++i) {
            const int mb = pr * 2 + i;
            const u32x4 a = av[q & 1][i];
#pragma unroll
            for (int b = 0; b < TNB; ++b) tot[mb][b] = mfma_bf16(a, bv[b], tot[mb][b]);
            if constexpr (GM == GM_G64) xs[mb] = mfma_bf16(a, __builtin_bit_cast(bf16x8, ones), J % 2 == 0 ? zero : xs[mb]);
            // Ones first: column lr of the result, in every register, is the sum of the block's row lr.
            else if (mb < OWN) xs_own[mb] = mfma_bf16(ones, __builtin_bit_cast(bf16x8, a), xs_own[mb]);
          }
          __builtin_amdgcn_sched_barrier(0);
        }
        if constexpr (GM == GM_G64 && J % 2 == 1) {    // leaving a group: remove offset and zero-point
          __builtin_amdgcn_sched_barrier(0);
          __builtin_amdgcn_s_setprio(0);
          float o[NC];
          spread(BASE + CM * float((szr[p][2] >> (zp_shift + 8 * G)) & 0xffu), o);
#pragma unroll
          for (int b = 0; b < TNB; ++b)
#pragma unroll
            for (int mb = 0; mb < TMB; ++mb)
#pragma unroll
              for (int r = 0; r < 4; ++r) tot[mb][b][r] -= o[b] * xs[mb][r];
        }
      };
      do_j(std::integral_constant<int, 0>{});
      do_j(std::integral_constant<int, 1>{});
      if constexpr (HALVES) {
        issue_half(0, kt + 1);
        fence(4, 8);
      }
      do_j(std::integral_constant<int, 2>{});
      do_j(std::integral_constant<int, 3>{});
      if constexpr (HALVES) issue_half(1, kt + 1);
    }
  };

  // factor that turns the accumulator into the result; per-channel scales are requested here, ahead of the main
  // loop (these formats have no group scales in flight, so the registers are there but for the larger codes of the large tile), instead of at its end.
  constexpr bool FIN_EARLY = GM == GM_PC && !CONV && (FMT == FMT_N4 || DIRECT);
  float fin[NC];
  auto load_fin = [&]() {
#pragma unroll
    for (int c = 0; c < NC; ++c)
      fin[c] = ncol(c) < ga.n ? reinterpret_cast<const __attribute__((address_space(1))) float*>(glb_bytes(blob[M32 ? 2 * c : c]) + ex.scale_off)[ncol(c)] : 1.f;
  };
  if constexpr (FIN_EARLY) load_fin();

  // ---- prologue: k-step 0 of the activations on its way to LDS, two weight steps in flight, requested in the order a step of
  // the loop leaves them: the loop's waits are counts of requests in flight, fixed at compile time for both ways into its head.
  // (Four staged k-steps instead of two: no faster on grids that fill a fraction of the chip, where one wave per SIMD is bound by
  // its own instructions, 1.2 us a k-step of the narrow tile, and 5 - 15 % slower on others.)
  if constexpr (EARLY) a_prepare();
  a_fetch(0, sh.buf[0]);
  __builtin_amdgcn_sched_barrier(0);
  if constexpr (DIRECT) fill_rows();                 // read in the epilogue and, the cleared sums, in the first k-step: behind the barrier below
  if constexpr (HALVES) { issue_half(0, 0); issue_half(1, 0); }
  else issue_w(1, 1);
  __builtin_amdgcn_sched_barrier(0);
  if constexpr (EARLY) a_prepare();
  wait_vm_lds<W_LOADS>();
  group_barrier();

  // ---- main loop, two k-steps per iteration so that ring slot and LDS buffer are static ----------
  auto step = [&](int kt, int p) {
    // the next step's activations, asked for as soon as this one's first reads of LDS are on their way; that buffer was last read in step kt - 1
    compute(p, kt, sh.buf[p], [&]() { a_fetch(kt + 1, sh.buf[p ^ 1]); });
    __builtin_amdgcn_sched_barrier(0);
    if constexpr (!HALVES) issue_w(p, kt + 2);
    __builtin_amdgcn_sched_barrier(0);
    if constexpr (EARLY) a_prepare();
    wait_vm_lds<W_LOADS>();                          // only the weights just requested may still be on their way
    group_barrier();
  };
  int kt = 0;
#pragma unroll 1
  for (; kt + 2 <= KT; kt += 2) {
    step(kt, 0);
    step(kt + 1, 1);
  }
  if constexpr (FULL) {
    lane = lane_here();
    lr = lane & 15;
    lq = lane >> 4;
  }
  if (kt < KT) compute(0, kt, sh.buf[0], [] {});     // uniform over the grid
  __builtin_amdgcn_sched_barrier(0);
  if constexpr (GM == GM_PC && !A8) {
    if (lq == 0) {
#pragma unroll
      for (int i = 0; i < OWN; ++i) sh.xs[(wave * OWN + i) * 16 + lr] = xs_own[i][0];
    }
  }
  wait_vm_lds<0>();
  group_barrier();

  // ---- epilogue -----------------------------------------------------------------------------------------
  if constexpr (GM != GM_PC) {
    spread(s_cur * INV_CM, fin);
  } else if constexpr (!FIN_EARLY) {
    load_fin();
  }
  float o_fin[NC];
  if constexpr (GM == GM_G128) spread(o_last, o_fin);
  // Weight rows outside the matrix are not stored.  Whole tiles of 16 are missing: a uniform branch, but for a block of 32 that is only half there.
  int col[NC];
  bool all[NC], some[NC];
#pragma unroll
  for (int c = 0; c < NC; ++c) {
    const int last = M32 && !MIXED ? 2 * c + 1 : c;
    col[c] = ncol(c);
    all[c] = (ntile * TWAVES + wave) * HB + last % HB < NT;
    some[c] = M32 && col[c] < ga.n;
  }
  auto put = [&](int c, auto* at, auto v) {
    if (all[c]) *at = v;
    else if (M32 && some[c]) *at = v;
  };
#pragma unroll
  for (int q = 0; q < NQ; ++q) {
    const int row0 = quad_row(q);
    f32x4 xs4 = {0.f, 0.f, 0.f, 0.f}, sx4 = xs4;
    if constexpr (GM == GM_G128) xs4 = *reinterpret_cast<const f32x4*>(sh.xs + ((KT - 1) & 1) * TBM_MAX + row0);      // the last group's row sums
    if constexpr (GM == GM_PC && !A8) xs4 = *reinterpret_cast<const f32x4*>(sh.xs + row0);
    if constexpr (A8) sx4 = *reinterpret_cast<const f32x4*>(sh.sx + row0);
    const i32x4 drow4 = *reinterpret_cast<const i32x4*>(sh.drow + row0);
    auto value = [&](int r, int c) {
      const float t = res(q, c, r);
      if constexpr (A8) return float(__float_as_int(t)) * sx4[r] * fin[c];
      else if constexpr (GM == GM_PC) return (fin[c] * INV_CM) * (t - off_sym * xs4[r]);
      else if constexpr (GM == GM_G128) return (t - o_fin[c] * xs4[r]) * fin[c];
      else return t * fin[c];
    };
    if constexpr (MIXED) {
      // Gate and up of a feature are 16 lanes apart: the even rows of 16 lanes take the gate and up values of result rows 0 and 1, the odd ones of 2 and 3.
#pragma unroll
      for (int r = 0; r < 2; ++r) {
        const auto v = __builtin_amdgcn_permlane16_swap(__float_as_uint(value(r, 0)), __float_as_uint(value(r + 2, 0)), false, false);
        const int drow = lq & 1 ? drow4[r + 2] : drow4[r];
        if (drow >= 0)
          put(0, static_cast<uint16_t*>(ga.y) + size_t(drow) * size_t(ga.n) + col[0], float_to_bf16_rne(silu_mul(__uint_as_float(v[0]), __uint_as_float(v[1]))));
      }
    } else {
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        if (drow4[r] >= 0) {
          float val[NC];
#pragma unroll
          for (int c = 0; c < NC; ++c) val[c] = value(r, c);
          const size_t drow = size_t(drow4[r]);
          if constexpr (GATEUP) {
            uint16_t* h = static_cast<uint16_t*>(ga.y) + drow * size_t(ga.n);
#pragma unroll
            for (int c = 0; c < NC / 2; ++c)
              put(c, h + col[c], float_to_bf16_rne(silu_mul(val[c], val[c + NC / 2])));
          } else if (ga.y_bf16) {
            uint16_t* y = static_cast<uint16_t*>(ga.y) + drow * size_t(ga.n);
#pragma unroll
            for (int c = 0; c < NC; ++c)
              put(c, y + col[c], float_to_bf16_rne(val[c]));
          } else {
            float* y = static_cast<float*>(ga.y) + drow * size_t(ga.n);
#pragma unroll
            for (int c = 0; c < NC; ++c)
              put(c, y + col[c], val[c]);
          }
        }
      }
    }
  }
}

// A launch with fewer than 8 weight tiles makes the patch narrower (2^patch_n_log2 weight tiles), so no
// work-group is launched for weight tiles that do not exist, and consecutive groups of PATCH_M row
// tiles still go round the XCDs.  Row tiles are enumerated expert by expert in the order of
// `TileGeom::order` (formats with the most arithmetic per tile first: what runs last, when the chip
// drains, are the cheap tiles).
constexpr int PATCH_M = 8;

template <int TMB, int TNB, bool GATEUP, bool CONV>
static __device__ __forceinline__ void tile_dispatch(const GemmArgs& ga, const TileGeom& tg, const ExpertDev& ex, const int off_e,
                                                     const int M_e, const int m0, const int ntile, const int wave, const TileLds& sh) {
  switch (ex.fmt * 4 + ex.gm) {
    case FMT_I8 * 4 + GM_PC: tile_task<TMB, TNB, FMT_I8, GM_PC, GATEUP, CONV>(ga, tg, ex, off_e, M_e, m0, ntile, wave, sh); break;
    case FMT_I8A8 * 4 + GM_PC:
      if constexpr (!CONV) tile_task<TMB, TNB, FMT_I8A8, GM_PC, GATEUP, CONV>(ga, tg, ex, off_e, M_e, m0, ntile, wave, sh);   // conv experts take bf16 rows
      break;
    case FMT_N6 * 4 + GM_PC:
      if constexpr (TMB == 4) tile_task<4, TNB, FMT_N6, GM_PC, GATEUP, CONV>(ga, tg, ex, off_e, M_e, m0, ntile, wave, sh);
      break;
    case FMT_N4 * 4 + GM_PC: tile_task<TMB, TNB, FMT_N4, GM_PC, GATEUP, CONV>(ga, tg, ex, off_e, M_e, m0, ntile, wave, sh); break;
    case FMT_N4 * 4 + GM_G128: tile_task<TMB, TNB, FMT_N4, GM_G128, GATEUP, CONV>(ga, tg, ex, off_e, M_e, m0, ntile, wave, sh); break;
    case FMT_N4 * 4 + GM_G64:
      if constexpr (TMB == 4) tile_task<4, TNB, FMT_N4, GM_G64, GATEUP, CONV>(ga, tg, ex, off_e, M_e, m0, ntile, wave, sh);
      break;
    case FMT_N3 * 4 + GM_G128: tile_task<TMB, TNB, FMT_N3, GM_G128, GATEUP, CONV>(ga, tg, ex, off_e, M_e, m0, ntile, wave, sh); break;
    case FMT_N3 * 4 + GM_G64:
      if constexpr (TMB == 4) tile_task<4, TNB, FMT_N3, GM_G64, GATEUP, CONV>(ga, tg, ex, off_e, M_e, m0, ntile, wave, sh);
      break;
    default: break;
  }
}

// Registers: the 128 x 256 tiles take all 256, nothing is spilled (see lane_here()).
template <bool GATEUP, bool CONV, int TNB>
__global__ __launch_bounds__(TWAVES * 64, TNB == 4 ? 2 : 3) void k_qgemm_tile(const GemmArgs ga, const TileGeom tg) {
  constexpr int MAX_ROWS = TNB == 4 && !CONV ? TBM_MAX : 64;
  constexpr int T_BUF = MAX_ROWS * 256;                // LDS bytes of one staged k-step
  constexpr int NROWS = TWAVES * TNB * 16 / (GATEUP ? 2 : 1);          // weight rows (of each matrix) per tile
  __shared__ __align__(1024) uint8_t buf0[T_BUF], buf1[T_BUF];     // two objects, so that the compiler can tell a buffer being filled from the one being read
  __shared__ __align__(16) float xs[2 * TBM_MAX];
  __shared__ __align__(16) int32_t drow[TBM_MAX];
  __shared__ __align__(16) float sx[TBM_MAX];
  __shared__ uint32_t src[TBM_MAX];
  __shared__ uint16_t taps[CONV ? TBM_MAX : 1];
  const TileLds sh{{buf0, buf1}, xs, drow, sx, src, taps};
  const int n_tiles = (ga.n + NROWS - 1) / NROWS;
  const int pn_log2 = tg.patch_n_log2, patch_wgs = PATCH_M << pn_log2;
  const int patches_n = (n_tiles + (1 << pn_log2) - 1) >> pn_log2;
  const int id = blockIdx.x, xcd = id & 7, j = id >> 3;
  const int patch = (j / patch_wgs) * 8 + xcd, q = j % patch_wgs;
  const int ntile = ((patch % patches_n) << pn_log2) + q / PATCH_M;
  if (ntile >= n_tiles) return;               // uniform over the work-group
  // Which expert and which row tile of its bucket: `slot` counts row tiles over all experts in the launch's
  // order.  Lane i takes the expert at position i: one load of the offsets, a prefix sum over 16 lanes.
  const int slot = (patch / patches_n) * PATCH_M + q % PATCH_M;
  const int lane = threadIdx.x & 63;
  const int mine = int((tg.order_bits >> (4 * (lane & 15))) & 15u);
  int o0 = 0, o1 = 0;
  if (lane < ga.n_experts) { o0 = ga.offsets[mine]; o1 = ga.offsets[mine + 1]; }
  int rows = (o1 - o0) * ga.T;
  if (rows < ga.min_rows || rows > ga.max_rows) rows = 0;         // that bucket belongs to the streaming kernel's launch
  // groups of 64 always take the small tile (their row sums are needed twice a k-step, by the wave itself), and so do 6-bit codes
  // (24 registers of codes too many: spills made the large tile the slower one)
  const int tbm = lane < ga.n_experts && (ga.ex[mine].gm == GM_G64 || ga.ex[mine].fmt == FMT_N6) ? 64 : tg.tbm;
  const int tiles = (rows + tbm - 1) / tbm;
  int incl = tiles;
#pragma unroll
  for (int d = 1; d < MOQE_MAX_EXPERTS; d <<= 1) {
    const int v = __shfl_up(incl, d);
    if (lane >= d) incl += v;
  }
  const unsigned long long hit = __ballot(lane < ga.n_experts && slot >= incl - tiles && slot < incl);
  if (hit == 0ull) return;                    // uniform: a surplus work-group
  const int at = __ffsll(hit) - 1;
  const int e = __builtin_amdgcn_readfirstlane(__shfl(mine, at));
  const int off_e = __builtin_amdgcn_readfirstlane(__shfl(o0, at));
  const int M_e = __builtin_amdgcn_readfirstlane(__shfl((o1 - o0) * ga.T, at));
  const int m0 = __builtin_amdgcn_readfirstlane(__shfl((slot - (incl - tiles)) * tbm, at));
  const int tbm_e = __builtin_amdgcn_readfirstlane(__shfl(tbm, at));
  const ExpertDev& ex = ga.ex[e];
  const int wave = TNB == 4 && !CONV ? __builtin_amdgcn_readfirstlane(int(threadIdx.x) >> 6) : 0;
  // a bucket's last tile with at most 64 rows left takes the small tile
  if constexpr (TNB == 4 && !CONV) {
    if (tbm_e == TBM_MAX && M_e - m0 > 64) {
      tile_dispatch<8, TNB, GATEUP, CONV>(ga, tg, ex, off_e, M_e, m0, ntile, wave, sh);
      return;
    }
  }
  tile_dispatch<4, TNB, GATEUP, CONV>(ga, tg, ex, off_e, M_e, m0, ntile, wave, sh);
}

// Relative arithmetic per tile of a format (measured on one launch per format): only the order matters.
static int tile_cost(const ExpertDev& ex) {
  const bool g64 = ex.gm == GM_G64, grp = ex.gm != GM_PC;
  switch (ex.fmt) {
    case FMT_I8A8: return 60;
    case FMT_I8:   return 119;
    case FMT_N6:   return 134;
    case FMT_N4:   return g64 ? 166 : (grp ? 125 : 108);
    default:       return g64 ? 172 : (grp ? 131 : 114);      // FMT_N3
  }
}

// The tile of a launch.
//  * 128 x 256 needs the least vector work per matrix operation and pays once its work-groups fill the chip: 8192 rows, K = 4, k 4096, n
//    4096: 286 us against 299 (64 x 256) and 307 (64 x 128).
//  * 64 x 128, three work-groups to a CU, fills places that 64 x 256 would leave empty: 1024 rows, n 11008: 144 us against 171; 1024
//    rows, n 4096: 57 against 73; 512 rows, n 1024: 40 against 50.
//  * 64 x 256 in between, two to a CU: 2048 rows, n 11008: 231 us against 243 (64 x 128) and 297 (128 x 256).
// Where the lines lie is a matter of rounds, and of the XCD that gets the most: a patch of tiles goes to one XCD, and few patches do not
// divide by eight (512 rows, n 11008: 11 patches of narrow tiles, two on three of the XCDs).  So the launch is laid out as the kernel lays
// it out, with the row tiles the buckets are expected to have, and timed: `t[i]` is the time of i + 1 work-groups sharing a CU, in units of
// one 64 x 256 tile alone, and about half each of the fullest XCD's time and of the chip's mean count.  The numbers were fitted to 1116
// launches (every format, K 1 to 16, even and skewed, 40 to 9000 rows, k 256 to 18944, n 256 to 11200) of this kernel before it had 32 x 32 x 16 products and
// priorities; on 420 other, random ones it then took 0.6 % longer than the best shape on average and 17 % at most (lines on the number of tiles 4 % and 54 %).  As
// the kernel is now: 1.2 % on average over 1979 launches, more than 5 % for one in eleven, 36 % at most.  Not fitted again.
// `equal`: every expert gets S / K samples (the label pass), so the row tiles are known; the half tile per bucket that an estimate adds
// starts a round that does not come (512 rows for each of four, k 11008, n 4096: 64 x 128; the whole pass 684 us instead of 646 with 64 x 256).
// `large_ok`: fewer than half of the experts have a format that stays at 64 rows (with two of three, int8 / int4 g64 / int3 g64, 6600 rows, n
// 2048: 140 us against 120), and it is no convolution, whose gather exists for 64 rows (128 x 256 spills; 128 x 128 would fit, not built).
enum TileShape { TILE_64x128, TILE_64x256, TILE_128x256 };
constexpr int XCDS = 8, CUS = 32;                                        // CUS: of one XCD
// Work-groups per CU of `rows` row tiles x `cols` weight tiles: of the fullest XCD, and on average.
struct Fill { float most, mean; };
static Fill fill(float rows, int cols) {
  int pn = 1;
  while (pn < cols && pn < 8) pn <<= 1;
  float load[XCDS] = {}, all = 0.f;
  int patch = 0;
  for (float left = rows; left > 0.f; left -= PATCH_M)
    for (int c = 0; c < cols; c += pn, ++patch) {
      const float wgs = std::min(left, float(PATCH_M)) * float(std::min(pn, cols - c));
      load[patch % XCDS] += wgs;
      all += wgs;
    }
  return {*std::max_element(load, load + XCDS) / CUS, all / float(XCDS * CUS)};
}
static float tile_time(float rows, int cols, int places, const float* t) {
  const auto [most, mean] = fill(rows, cols);
  const int full = int(most / float(places)), i = int(most - float(full * places));
  const float rest = most - float(full * places + i), lo = i ? t[i - 1] : 0.f;
  const float last = full ? lo + (t[i] - lo) * rest : t[i - (i && rest <= 0.05f ? 1 : 0)];
  return 0.53f * (float(full) * t[places - 1] + last) + 0.47f * mean / float(places) * t[places - 1];
}
// Row tiles that the buckets are expected to have: 64-row ones, and of the large shape 128-row ones and what is left as 64-row ones.
struct RowTiles { float r64, large, small; bool known; };
static RowTiles row_tiles(int M, int S, int T, int K, bool equal) {
  const int B = std::min(K, S);                                             // most buckets with rows
  // a bucket ends anywhere in its last tile, or on a multiple of T; the large tile's last 64 rows or less are a small one
  float r64 = T % 64 == 0 ? float(M / 64) : std::max(float(B), float(M) / 64.f + 0.5f * float(B - 1));
  float large = float(M) / 128.f, small = T % 128 == 0 ? 0.f : 0.5f * float(B);
  if (T % 64 == 0) large -= 0.5f * small;
  const bool known = B == 1 || equal;                                      // the rows of each bucket
  if (known) {
    const int n_b = equal ? K : 1, m = M / n_b;
    r64 = float(n_b * ((m + 63) / 64));
    large = float(n_b * (m / 128 + (m % 128 > 64))); small = m % 128 > 0 && m % 128 <= 64 ? float(n_b) : 0.f;
  }
  return {r64, large, small, known};
}
static TileShape tile_shape(const RowTiles& rt, int M, int n, int wide_n, bool large_ok) {
  const int wide = (n + wide_n - 1) / wide_n, narrow = (n + wide_n / 2 - 1) / (wide_n / 2);
  if (long(M / 128) * wide >= 4096) return large_ok ? TILE_128x256 : TILE_64x256;     // eight rounds and more
  static const float t_narrow[3] = {0.28f, 0.5f, 0.91f}, t_wide[2] = {1.f, 1.14f}, t_large[2] = {1.76f, 2.08f};
  const float a = tile_time(rt.r64, narrow, 3, t_narrow), b = tile_time(rt.r64, wide, 2, t_wide);
  if (large_ok) {
    const float c = tile_time(rt.large + rt.small, wide, 2, t_large) * (1.f - 0.175f * rt.small / (rt.large + rt.small));    // a launch of small tiles alone would take a sixth less here
    if (c < std::min(a, b)) return TILE_128x256;
  }
  return a <= b ? TILE_64x128 : TILE_64x256;
}

// Products ahead of the other work-groups' rescaling and unpacking (raise_priority()), but for launches whose last round is a few work-groups or at most one for a
// CU.  Priorities keep the work-groups of a CU out of step (whole rounds of 128 x 256 tiles take 1.00 - 1.18 times as long without), and a CU that is early then takes
// two of the last round's while another gets none.  Time without / with priorities, launches of two to eight experts:
//  * 128 x 256, the buckets' rows known (260 label passes), by rounds of the fullest XCD: 1.06 - 1.5 0.83 - 1.00 (mean 0.91), 2.06 - 2.5 0.92 - 0.99, 3.06 - 3.5
//    0.94 - 1.01, 4.06 - 4.5 0.96 - 1.015, 5.5 0.99, more 0.98 - 1.02; with three quarters of a last round 1.02 - 1.04.
//  * Routed batches (1700 launches) end anywhere around the expected number of tiles, so the chip's mean counts: up to an eighth past one to four rounds 0.97,
//    0.95, 0.97 and 0.985 on average (8192 rows in four buckets, k and n 4096: 288 us against 326), further on 0.99 - 1.07.  64 x 256: up to a twelfth past two and three
//    0.98, else 0.98 - 1.14.
//  * 64 x 128, three to a CU: one more work-group for each (1.05 to 1.38 rounds of the fullest XCD) 0.97, 1.3 to 1.38 0.96; else 0.99 - 1.13.
static bool products_first(const RowTiles& rt, TileShape shape, int n, int wide_n) {
  const bool narrow = shape == TILE_64x128, large = shape == TILE_128x256;
  const int cols = narrow ? (n + wide_n / 2 - 1) / (wide_n / 2) : (n + wide_n - 1) / wide_n;
  const float tiles = large ? rt.large + rt.small : rt.r64;
  if (tiles * float(cols) >= 4096.f) return true;
  const auto [most, mean] = fill(tiles, cols);
  if (narrow) return most < 3 * 1.05f || most > 3 * 1.38f;
  const float rounds = (rt.known ? most : mean) / 2.f, last = rounds - std::floor(rounds);
  if (rt.known) return !(large && rounds >= 1.f && rounds < 6.f && last > 0.06f && last < 0.55f);
  return !(rounds >= (large ? 1.f : 2.f) && rounds < (large ? 5.f : 4.f) && last > 0.01f && last < (large ? 0.13f : 0.08f));
}

int32_t launch_qgemm_tile(const GemmArgs& ga, bool gateup, bool equal, hipStream_t st) {
  const int M = ga.S * ga.T;
  TileGeom tg;
  memset(&tg, 0, sizeof(tg));
  int low = 0;                                                          // experts that take 64 rows in any case
  for (int e = 0; e < ga.n_experts; ++e) low += ga.ex[e].gm == GM_G64 || ga.ex[e].fmt == FMT_N6;
  const int wide_n = gateup ? 128 : 256;                               // weight rows of the wide tiles
  const RowTiles rt = row_tiles(M, ga.S, ga.T, ga.n_experts, equal);
  const TileShape shape = tile_shape(rt, M, ga.n, wide_n, ga.conv_c == 0 && 2 * low < ga.n_experts);
  const bool wide_tile = shape != TILE_64x128;
  tg.products_first = products_first(rt, shape, ga.n, wide_n) ? 1 : 0;
  tg.tbm = shape == TILE_128x256 ? TBM_MAX : 64;
  const int least = low > 0 ? 64 : tg.tbm;                                  // height of the lowest tiles in the launch
  const int row_tiles = (M + least - 1) / least + ga.n_experts;         // upper bound on sum_e ceil(M_e / tbm_e)
  const int n_rows = wide_tile ? wide_n : wide_n / 2;
  const int n_tiles = (ga.n + n_rows - 1) / n_rows;
  tg.a_bytes = uint32_t(size_t(M) * size_t(ga.conv_c > 0 ? ga.conv_c : ga.k) * 2);
  while ((1 << tg.patch_n_log2) < n_tiles && tg.patch_n_log2 < 3) ++tg.patch_n_log2;
  const int pn = 1 << tg.patch_n_log2;
  const long patches = long((row_tiles + PATCH_M - 1) / PATCH_M) * ((n_tiles + pn - 1) / pn);
  const long grid = (patches + 7) / 8 * 8 * (PATCH_M * pn);
  if (grid > 0x7fffffffL) return set_error(MOQE_E_SHAPE, "grouped_qgemm: %d rows exceed the tile kernel's grid", M);
  static_assert(MOQE_MAX_EXPERTS <= 16, "the order is packed in 4-bit fields");
  int order[MOQE_MAX_EXPERTS];
  for (int e = 0; e < ga.n_experts; ++e) order[e] = e;
  std::stable_sort(order, order + ga.n_experts, [&](int a, int b) { return tile_cost(ga.ex[a]) > tile_cost(ga.ex[b]); });
  for (int e = 0; e < ga.n_experts; ++e) tg.order_bits |= uint64_t(order[e]) << (4 * e);
  const bool conv = ga.conv_c > 0;
  if (conv) {
    if (ga.conv_c % 128 != 0 || ga.conv_c > 16384) return set_error(MOQE_E_SHAPE, "grouped_qgemm: the convolution gather takes 128 to 16384 input channels in multiples of 128, not %d", ga.conv_c);
  }
  ProfileScope ps(gateup ? MOQE_PK_GEMM_GATEUP : MOQE_PK_GEMM_PLAIN, st, true);
  const dim3 g{unsigned(grid), 1, 1}, t{TWAVES * 64, 1, 1};
  auto go = [&](auto kernel_gateup, auto kernel_conv, auto kernel_plain) {
    if (gateup) ps.launch(kernel_gateup, g, t, 0, ga, tg);
    else if (conv) ps.launch(kernel_conv, g, t, 0, ga, tg);
    else ps.launch(kernel_plain, g, t, 0, ga, tg);
  };
  if (wide_tile) go(k_qgemm_tile<true, false, 4>, k_qgemm_tile<false, true, 4>, k_qgemm_tile<false, false, 4>);
  else go(k_qgemm_tile<true, false, 2>, k_qgemm_tile<false, true, 2>, k_qgemm_tile<false, false, 2>);
  return check_launch("grouped_qgemm(tile)");
}

}  // namespace moqe
