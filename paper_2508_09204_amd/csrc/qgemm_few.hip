// Grouped dequantize-GEMM for launches of at most 16 rows in all (one request being decoded, or a few).
//
// Each sample is processed by its selected expert only (MoQE Section 3.1): with so few samples few experts have a bucket, of a row or
// two, and the launch is one pass over those experts' packed weights.  What bounds it is how soon, and by how many waves, the weights
// are asked for.  Hence a work-group per 16 weight rows (gate/up: 16 rows of each) of the experts that CAN have rows - at most one
// per sample, found on the device - whose waves (four for gate/up, eight for a plain product) share the k-tiles out among them and keep two
// in flight each.  A wave reads its activation
// operands straight into registers, 16 bytes per lane of the row it stands for (rows past the bucket repeat its last one): there is
// no staging, and no barrier before the one ahead of the sum over the waves.  Arithmetic as in qgemm_stream_lds.hip: exact codes on
// the bf16 matrix cores, offset and zero-point removed with the row sums, fp32 scale per group.
// Blocks of 4096 / 11008, K = 4 (int4, int4, int3, int8), against the streaming kernels (a persistent schedule; 64 work-groups per expert for long
// rows): one token 45 -> 33 us where it goes to an int4 expert, 49 -> 33 int3, 54 -> 39 int8, S = 2 68 -> 57, S = 4 90 -> 87, S = 16 90 -> 90;
// 3584 / 18944, K = 8, S = 16 242 -> 232; 512 / 16384, K = 3, S = 1 47 -> 21.  Launches of many work-groups are the streaming kernels':
// few_rows_kernel() in dispatch_rules.h.
#include "dispatch_rules.h"
#include "qgemm_device.h"
#include "self_bucket.h"

namespace moqe {

namespace few {
constexpr int PART = 4 * 64;                     // floats of a wave's 16 x 16 partial result
// Waves of a work-group.  Rows of the gate and up matrices are short (32 k-tiles of 4096 columns) and there are many: four waves, four
// work-groups to a CU, take what eight waves would in a second round (S = 1, 4096 / 11008: the block 44.2 us with four against 46.8
// with eight and 49.5 with sixteen, down projection by qgemm_stream_lds.hip).  A down projection has few and long rows: eight (with
// four the block takes 35.8 us, eight 34.3, sixteen 34.4).
constexpr int waves(bool gateup) { return gateup ? 4 : 8; }

template <int FMT, int GM, bool GATEUP>
static __device__ __forceinline__ void few_task(const GemmArgs& ga, const ExpertDev& ex, const int off_e, const int M_e, const int nt,
                                                float* part, const int32_t* perm_l) {
  constexpr bool A8 = (FMT == FMT_I8A8);
  constexpr int NS = GATEUP ? 2 : 1, WAVES = waves(GATEUP);
  constexpr int NR = Raw<FMT>::N;
  constexpr int GPT = GM == GM_PC ? 0 : (GM == GM_G128 ? 1 : 2);
  constexpr int AJ = A8 ? 2 : 4;                 // matrix-core steps per k-tile
  // k-tiles in flight.  Two fit 128 registers, with which 16 waves share a CU; four and half the waves are slower (the block at S = 1
  // 35.8 -> 40.3 us, at S = 4 84 -> 115: the set-up of one work-group has to run beside another's loads).
  constexpr int PF = 2;
  constexpr float BASE = CodeMap<FMT>::BASE, CM = CodeMap<FMT>::CM, INV_CM = 1.f / CodeMap<FMT>::CM;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int lr = lane & 15, lq = lane >> 4;
  const int KT = ga.k >> 7, T = ga.T;
  const FragK<FMT> fk = frag_constants<FMT>();
  const u32x4 ones = {0x3F803F80u, 0x3F803F80u, 0x3F803F80u, 0x3F803F80u};
  const bf16x8 ones_b = __builtin_bit_cast(bf16x8, ones);
  const f32x4 zero = {0.f, 0.f, 0.f, 0.f};

  // ---- rings: tile i of this wave is k-tile wave + WAVES i
  const buf_rsrc rsrc[2] = {blob_rsrc(ex.w[0]), blob_rsrc(ex.w[GATEUP ? 1 : 0])};
  const uint32_t t0 = uint32_t(nt) * uint32_t(KT);
  const int n_it = wave < KT ? (KT - wave + WAVES - 1) / WAVES : 0;
  uint32_t raw[PF][NS][NR];
  float sc[PF][NS][GPT ? GPT : 1];
  uint16_t zp[PF][NS];
  u32x4 av[PF][AJ];
  auto issue_w = [&](int p, int i) {
    const uint32_t t = t0 + uint32_t(min(wave + WAVES * i, KT - 1));
#pragma unroll
    for (int s = 0; s < NS; ++s) {
      load_raw<FMT>(raw[p][s], rsrc[s], t * ex.tile_bytes, lane);
      if constexpr (GPT == 1) {
        sc[p][s][0] = __uint_as_float(buf_load32(rsrc[s], lr * 4, ex.scale_off + t * 64u));
        zp[p][s] = uint16_t(__builtin_amdgcn_raw_buffer_load_b8(rsrc[s], lr, int(ex.zero_off + t * 16u), 0));
      } else if constexpr (GPT == 2) {
        const u32x2 v = buf_load64(rsrc[s], lr * 8, ex.scale_off + t * 128u);
        sc[p][s][0] = __uint_as_float(v.x); sc[p][s][GPT - 1] = __uint_as_float(v.y);
        zp[p][s] = uint16_t(__builtin_amdgcn_raw_buffer_load_b16(rsrc[s], lr * 2, int(ex.zero_off + t * 32u), 0));
      }
    }
  };
  // the first weights are on their way before the rows are looked up
#pragma unroll
  for (int p = 0; p < PF; ++p) issue_w(p, p);
  __builtin_amdgcn_sched_barrier(0);
  uint32_t a_off;                                // byte offset of this lane's share of its row (< 4 GiB, checked before the launch)
  {
    const int m = min(lr, M_e - 1);
    int row = off_e * T + m;
    if constexpr (!A8) {
      if (ga.a_perm) {
        const int q = T == 1 ? m : m / T, smp = perm_l ? perm_l[off_e + q] : ga.a_perm[off_e + q];
        row = smp * T + (m - q * T);
      }
    }
    a_off = uint32_t(row) * uint32_t(ga.k) * (A8 ? 1u : 2u) + uint32_t(lq) * 16u;
  }
  const buf_rsrc a_rsrc = blob_rsrc(reinterpret_cast<const uint8_t*>(A8 ? static_cast<const void*>(ga.a_q) : ga.a));
  auto issue_a = [&](int p, int i) {
    const uint32_t at = uint32_t(min(wave + WAVES * i, KT - 1)) * (A8 ? 128u : 256u);
#pragma unroll
    for (int j = 0; j < AJ; ++j) av[p][j] = buf_load128(a_rsrc, int(a_off), at + uint32_t(j) * 64u);
  };
#pragma unroll
  for (int p = 0; p < PF; ++p) issue_a(p, p);
  // what the epilogue needs: the sum over the waves is taken by the first four, wave r the rows 4 lq + r
  const int m_out = 4 * lq + wave;
  int out_row = off_e * T + m_out;
  float sx = 1.f, pcs[NS];
  if (wave < 4 && m_out < M_e) {
    if constexpr (A8) sx = ga.a_scale[out_row];
    if constexpr (!GATEUP) {
      if (ga.y_perm) {
        const int q = T == 1 ? m_out : m_out / T, smp = perm_l ? perm_l[off_e + q] : ga.y_perm[off_e + q];
        out_row = smp * T + (m_out - q * T);
      }
    }
  }
  if constexpr (GM == GM_PC) {
#pragma unroll
    for (int s = 0; s < NS; ++s) pcs[s] = __uint_as_float(buf_load32(rsrc[s], lr * 4, ex.scale_off + uint32_t(nt) * 64u));
  }
  __builtin_amdgcn_sched_barrier(0);

  f32x4 tot[NS], xs_tot = zero;                  // bf16 path: fp32 sums; int8 path: int32 bit patterns
#pragma unroll
  for (int s = 0; s < NS; ++s) tot[s] = zero;
  auto consume = [&](int p) {
    if constexpr (A8) {
#pragma unroll
      for (int s = 0; s < NS; ++s) {
        i32x4 acc = __builtin_bit_cast(i32x4, tot[s]);
#pragma unroll
        for (int j = 0; j < 2; ++j) {
          const i32x4 b = {int(raw[p][s][4 * j]), int(raw[p][s][4 * j + 1]), int(raw[p][s][4 * j + 2]), int(raw[p][s][4 * j + 3])};
          acc = __builtin_amdgcn_mfma_i32_16x16x64_i8(__builtin_bit_cast(i32x4, av[p][j]), b, acc, 0, 0, 0);
        }
        tot[s] = __builtin_bit_cast(f32x4, acc);
      }
    } else {
      const u32x4 a0 = av[p][0], a1 = av[p][1], a2 = av[p][AJ - 2], a3 = av[p][AJ - 1];
      f32x4 xs0 = GM == GM_PC ? xs_tot : zero, xs1 = zero;
      xs0 = mfma_bf16(a1, ones_b, mfma_bf16(a0, ones_b, xs0));
      if constexpr (GM == GM_G64) xs1 = mfma_bf16(a3, ones_b, mfma_bf16(a2, ones_b, zero));
      else xs0 = mfma_bf16(a3, ones_b, mfma_bf16(a2, ones_b, xs0));
      if constexpr (GM == GM_PC) xs_tot = xs0;
#pragma unroll
      for (int s = 0; s < NS; ++s) {
        const bf16x8 b0 = frag<FMT, 0>(raw[p][s], fk), b1 = frag<FMT, 1>(raw[p][s], fk), b2 = frag<FMT, 2>(raw[p][s], fk),
                     b3 = frag<FMT, 3>(raw[p][s], fk);
        if constexpr (GM == GM_PC) {
          tot[s] = mfma_bf16(a3, b3, mfma_bf16(a2, b2, mfma_bf16(a1, b1, mfma_bf16(a0, b0, tot[s]))));
        } else if constexpr (GM == GM_G128) {
          const f32x4 v = mfma_bf16(a3, b3, mfma_bf16(a2, b2, mfma_bf16(a1, b1, mfma_bf16(a0, b0, zero))));
          const float o = BASE + CM * float(uint32_t(zp[p][s]) & 0xffu), f = sc[p][s][0] * INV_CM;
#pragma unroll
          for (int r = 0; r < 4; ++r) tot[s][r] += f * (v[r] - o * xs0[r]);
        } else {
          const f32x4 v0 = mfma_bf16(a1, b1, mfma_bf16(a0, b0, zero)), v1 = mfma_bf16(a3, b3, mfma_bf16(a2, b2, zero));
          const float o0 = BASE + CM * float(uint32_t(zp[p][s]) & 0xffu), o1 = BASE + CM * float((uint32_t(zp[p][s]) >> 8) & 0xffu);
          const float f0 = sc[p][s][0] * INV_CM, f1 = sc[p][s][GPT == 2 ? 1 : 0] * INV_CM;
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            tot[s][r] += f0 * (v0[r] - o0 * xs0[r]);
            tot[s][r] += f1 * (v1[r] - o1 * xs1[r]);
          }
        }
      }
    }
  };
  int i = 0;
#pragma unroll 1
  for (; i + 2 * PF <= n_it; i += PF) {
#pragma unroll
    for (int p = 0; p < PF; ++p) {
      consume(p);
      issue_w(p, i + p + PF);
      issue_a(p, i + p + PF);
      __builtin_amdgcn_sched_barrier(0);
    }
  }
#pragma unroll
  for (int p = 0; p < 2 * PF - 1; ++p) {         // uniform over the wave: what is left, fewer than 2 PF tiles
    if (i + p < n_it) consume(p % PF);
    if (p < PF - 1 && i + p + PF < n_it) {
      issue_w(p, i + p + PF);
      issue_a(p, i + p + PF);
    }
    __builtin_amdgcn_sched_barrier(0);
  }

  // ---- the waves' shares, in wave order
  constexpr bool XS = GM == GM_PC && !A8;
  float* mine = part + wave * (NS + 1) * PART;
#pragma unroll
  for (int s = 0; s < NS; ++s)
#pragma unroll
    for (int r = 0; r < 4; ++r) mine[s * PART + r * 64 + lane] = tot[s][r];
  if constexpr (XS) {
#pragma unroll
    for (int r = 0; r < 4; ++r) mine[NS * PART + r * 64 + lane] = xs_tot[r];
  }
  __syncthreads();
  if (wave >= 4 || m_out >= M_e) return;
  float val[NS], xs = 0.f;
#pragma unroll
  for (int w = 0; w < WAVES; ++w) if constexpr (XS) xs += part[w * (NS + 1) * PART + NS * PART + tid];
#pragma unroll
  for (int s = 0; s < NS; ++s) {
    if constexpr (A8) {
      int v = 0;
#pragma unroll
      for (int w = 0; w < WAVES; ++w) v += __float_as_int(part[w * (NS + 1) * PART + s * PART + tid]);
      val[s] = float(v) * sx * pcs[s];
    } else {
      float v = 0.f;
#pragma unroll
      for (int w = 0; w < WAVES; ++w) v += part[w * (NS + 1) * PART + s * PART + tid];
      val[s] = v;
      if constexpr (GM == GM_PC) val[s] = (pcs[s] * INV_CM) * (v - (BASE + CM * float(ex.zc)) * xs);
    }
  }
  const size_t at = size_t(out_row) * size_t(ga.n) + nt * 16 + lr;
  if constexpr (GATEUP) static_cast<uint16_t*>(ga.y)[at] = float_to_bf16_rne(silu_mul(val[0], val[NS - 1]));
  else if (ga.y_bf16) static_cast<uint16_t*>(ga.y)[at] = float_to_bf16_rne(val[0]);
  else static_cast<float*>(ga.y)[at] = val[0];
}

}  // namespace few

// grid: x = tile of 16 weight rows, y = place among the experts that have rows, for as many as can have some.  (The gate/up instance spills one register, set up ahead of
// its loads.)
template <bool GATEUP>
__global__ __launch_bounds__(few::waves(GATEUP) * 64, 4) void k_qgemm_few(const GemmArgs ga) {
  __shared__ float part[few::waves(GATEUP) * (GATEUP ? 3 : 2) * few::PART];
  __shared__ int32_t perm[few::waves(GATEUP) * 64];
  const int lane = threadIdx.x & 63, K = ga.n_experts;
  // every lane's expert, requested together with what decides between them: read after the choice, the descriptor would be one more
  // dependent trip to memory before the first weight (2048 x 2048, one row: 4.5 us, with it 4.3)
  const ExpertDev mine = ga.ex[lane < K ? lane : 0];
  int o0 = 0, o1 = 0;
  int32_t* perm_l = nullptr;
  if (ga.expert_idx) {
    perm_l = perm + (threadIdx.x >> 6) * 64;
    self_bucket(ga, lane, o0, o1, perm_l, blockIdx.x == 0 && blockIdx.y == 0 && threadIdx.x < 64);
  } else if (lane < K) {
    o0 = ga.offsets[lane];
    o1 = ga.offsets[lane + 1];
  }
  unsigned long long busy = __ballot(lane < K && o1 > o0);
  for (int y = blockIdx.y; y > 0 && busy; --y) busy &= busy - 1;
  if (busy == 0ull) return;                      // uniform: fewer experts than the grid allows for
  const int e = __ffsll(busy) - 1;
  const int off_e = __builtin_amdgcn_readlane(o0, e);
  const int M_e = (__builtin_amdgcn_readlane(o1, e) - off_e) * ga.T;
  auto from_lane = [&](uint32_t v) { return uint32_t(__builtin_amdgcn_readlane(int(v), e)); };
  auto blob = [&](const uint8_t* p) {
    const uint64_t v = reinterpret_cast<uint64_t>(p);
    return reinterpret_cast<const uint8_t*>(uint64_t(from_lane(uint32_t(v >> 32))) << 32 | from_lane(uint32_t(v)));
  };
  ExpertDev ex;
  ex.w[0] = blob(mine.w[0]); ex.w[1] = blob(mine.w[1]);
  ex.fmt = int(from_lane(mine.fmt)); ex.gm = int(from_lane(mine.gm)); ex.zc = int(from_lane(mine.zc)); ex.asym = int(from_lane(mine.asym));
  ex.tile_bytes = from_lane(mine.tile_bytes); ex.scale_off = from_lane(mine.scale_off); ex.zero_off = from_lane(mine.zero_off);
  const int nt = blockIdx.x;
  switch (ex.fmt * 4 + ex.gm) {
    case FMT_I8 * 4 + GM_PC:     few::few_task<FMT_I8, GM_PC, GATEUP>(ga, ex, off_e, M_e, nt, part, perm_l); break;
    case FMT_I8A8 * 4 + GM_PC:   few::few_task<FMT_I8A8, GM_PC, GATEUP>(ga, ex, off_e, M_e, nt, part, perm_l); break;
    case FMT_N6 * 4 + GM_PC:     few::few_task<FMT_N6, GM_PC, GATEUP>(ga, ex, off_e, M_e, nt, part, perm_l); break;
    case FMT_N4 * 4 + GM_PC:     few::few_task<FMT_N4, GM_PC, GATEUP>(ga, ex, off_e, M_e, nt, part, perm_l); break;
    case FMT_N4 * 4 + GM_G128:   few::few_task<FMT_N4, GM_G128, GATEUP>(ga, ex, off_e, M_e, nt, part, perm_l); break;
    case FMT_N4 * 4 + GM_G64:    few::few_task<FMT_N4, GM_G64, GATEUP>(ga, ex, off_e, M_e, nt, part, perm_l); break;
    case FMT_N3 * 4 + GM_G128:   few::few_task<FMT_N3, GM_G128, GATEUP>(ga, ex, off_e, M_e, nt, part, perm_l); break;
    case FMT_N3 * 4 + GM_G64:    few::few_task<FMT_N3, GM_G64, GATEUP>(ga, ex, off_e, M_e, nt, part, perm_l); break;
    default: break;
  }
}

int32_t launch_qgemm_few(const GemmArgs& ga, bool gateup, hipStream_t st) {
  const int M = ga.S * ga.T;
  if (M > FEW_MAX_ROWS || ga.conv_c != 0) return set_error(MOQE_E_SHAPE, "grouped_qgemm: the kernel for few rows takes %d at most, not %d", FEW_MAX_ROWS, M);
  const dim3 g(unsigned(ga.n / 16), unsigned(ga.S < ga.n_experts ? ga.S : ga.n_experts)), t(few::waves(gateup) * 64);
  ProfileScope ps(gateup ? MOQE_PK_GEMM_GATEUP : MOQE_PK_GEMM_PLAIN, st, true);
  if (gateup) ps.launch(k_qgemm_few<true>, g, t, 0, ga);
  else ps.launch(k_qgemm_few<false>, g, t, 0, ga);
  return check_launch("grouped_qgemm(few)");
}

}  // namespace moqe
