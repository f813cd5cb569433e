// The NLP router model (MoQE Section 3.2): token vectors -> projection -> one post-norm Transformer encoder
// layer -> a second self-attention module (residual, LayerNorm) -> mean over the tokens -> MLP head -> top-1.
// The paper fixes the order of the stages, not their sizes; widths come with the parameter struct.
//
// Kernels of this file (router_nlp_rows.hip has those that take whole rows through several stages, for the usual widths and batches):
//   k_to_bf16      fp32 parameters -> bf16 copies (one launch for all matrices)
//   k_lin          C = A W^T + bias [+ residual] [ReLU] on the bf16 matrix cores, fp32 accumulation; A and W
//                  are bf16, C is written as fp32 and/or bf16
//   k_attention    softmax(Q K^T / sqrt(dh)) V per (sample, head), fp32 products from exact bf16 pieces, 16 queries per wave,
//                  keys streamed in tiles of 32 through LDS with a running maximum and sum; k_attention_fp32 for few tokens
//   k_layer_norm   per row, fp32, biased variance; writes fp32 and/or bf16
//   k_ln_pool      the last LayerNorm and the mean over a sample's tokens (k_pool_f32 adds the chunks of long samples)
// The MLP head on the pooled vector is the small router of route.hip.
#include "bf16_pieces.h"
#include "dispatch_rules.h"
#include "qgemm_device.h"

#include <algorithm>
#include <cstring>

namespace moqe {

// ---- parameters to bf16 ---------------------------------------------------------------------------------
constexpr int CVT_MAX_SEG = 8;
struct CvtSegs {
  const float* src[CVT_MAX_SEG];
  uint16_t* dst[CVT_MAX_SEG];
  long long first[CVT_MAX_SEG + 1];      // first[i] = index (in units of 4 elements) where segment i starts
  int n;
};

__global__ __launch_bounds__(256) void k_to_bf16(const CvtSegs sg) {
  const long long total = sg.first[sg.n];
  for (long long i = blockIdx.x * 256ll + threadIdx.x; i < total; i += gridDim.x * 256ll) {
    int s = 0;
#pragma unroll
    for (int j = 1; j < CVT_MAX_SEG; ++j) s += (j < sg.n && i >= sg.first[j]) ? 1 : 0;
    const long long e = (i - sg.first[s]) * 4;
    const float4 v = *reinterpret_cast<const float4*>(sg.src[s] + e);
    uint2 o;
    o.x = pack_bf16x2(v.x, v.y);
    o.y = pack_bf16x2(v.z, v.w);
    *reinterpret_cast<uint2*>(sg.dst[s] + e) = o;
  }
}

// ---- C = A W^T ---------------------------------------------------------------------------------------------
// Work-group tile 128 rows x 128 columns, k-tiles of 32; 4 waves as 2 x 2, a wave owns 64 x 64 (4 x 4 matrix-core blocks).  The products
// of a router are short (k = 384: 12 k-tiles), so what bounds them is filling and draining a tile: 32 KB of LDS and 100 registers let
// four work-groups share a CU and overlap.  Both operand tiles are loaded into LDS directly (rows of 64 bytes, 16-byte units
// XOR-swizzled by row / 4: the lane that fills a unit loads the swizzled column, and the operand reads of 16 rows meet 16 different
// bank quads), double-buffered, one barrier per k-tile.  Tiles of the same rows follow one another on the same XCD, whose L2 then
// reads the rows once (spread over the XCDs, 3584 -> 384 read its input three times).
// 32768 rows: 3584 -> 384 135 us, 384 -> 1152 81, 384 -> 384 57, 384 -> 1536 90, 1536 -> 384 84 with k-tiles of 64 through registers and
// two work-groups to a CU and stores
// straight from the accumulators; now 127, 51, 42, 60, 69.  (A third buffer, two k-tiles ahead: no faster, 144 us on the first.)
// NB = 4: four buffers, three k-tiles in flight, for launches of few work-groups (see LIN_DEEP_MAX).
constexpr int LBM = 128, LBN = 128, LBK = 32;
constexpr int L_TILE_BYTES = LBM * LBK * 2;                  // one operand tile

struct LinArgs {
  const uint16_t* a;      // bf16 [M, k]
  const uint16_t* w;      // bf16 [n, k]
  const float* bias;      // [n] or NULL
  const float* residual;  // fp32 [M, n] or NULL, added after the bias
  float* c32;             // fp32 [M, n] or NULL
  uint16_t* c16;          // bf16 [M, n] or NULL
  int M, n, k;
  int relu;
  int by_xcd;             // tiles of the same rows on the same XCD
  int ksplit;             // > 1: work-group z multiplies its share of the k-tiles and stores the raw sums to part[z]
  float* part;            // fp32 [ksplit, M, n]
};

typedef __attribute__((address_space(3))) void lds_ptr;

template <int NB>
__global__ __launch_bounds__(256, NB == 2 ? 4 : 2) void k_lin(const LinArgs la) {
  __shared__ __align__(1024) uint8_t buf0[2 * L_TILE_BYTES], buf1[2 * L_TILE_BYTES];   // A, then W; separate objects the compiler can tell apart
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int lr = lane & 15, lq = lane >> 4;
  const int wm = wave >> 1, wn = wave & 1;
  const int n_tiles = la.n / LBN, m_tiles = (la.M + LBM - 1) / LBM;
  // Work-groups go round the XCDs: id % 8.  Whole groups of eight row tiles give every XCD one of them; the rest go round tile by tile.
  const int id = blockIdx.x, dealt = la.by_xcd ? (m_tiles & ~7) : 0;
  const bool whole = id < dealt * n_tiles;
  const int j = whole ? id >> 3 : id - dealt * n_tiles;
  const int mt = whole ? (j / n_tiles) * 8 + (id & 7) : dealt + j / n_tiles;
  const int m0 = mt * LBM, n0 = (j % n_tiles) * LBN;
  const int KT = la.k / LBK;
  const int kt0 = int(blockIdx.z) * KT / la.ksplit, kt1 = (int(blockIdx.z) + 1) * KT / la.ksplit;   // this work-group's k-tiles
  // request i of a wave fills 1 KiB: rows 16 (4 i + wave) + lane / 4 of the tile; descriptors start at the tile's first row
  const uint32_t pitch = uint32_t(la.k) * 2u;
  const int rows_a = min(LBM, la.M - m0);
  const buf_rsrc a_rsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t*>(la.a + size_t(m0) * la.k), 0, uint32_t(rows_a) * pitch, 0x00020000);
  const buf_rsrc w_rsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t*>(la.w + size_t(n0) * la.k), 0, uint32_t(LBN) * pitch, 0x00020000);
  const int s_row = wave * 16 + (lane >> 2);
  const uint32_t s_col = uint32_t((lane & 3) ^ ((lane >> 4) & 3)) * 16u;      // (row >> 2) & 3 = (lane >> 4) & 3
  uint32_t a_off[2], w_off[2];
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    a_off[i] = uint32_t(min(s_row + 64 * i, rows_a - 1)) * pitch + s_col;     // rows past the end repeat the last row
    w_off[i] = uint32_t(s_row + 64 * i) * pitch + s_col;
  }
  auto fetch = [&](uint8_t* buf, int kt) {
    const int ko = min(kt, kt1 - 1) * (LBK * 2);
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      __builtin_amdgcn_raw_ptr_buffer_load_lds(a_rsrc, (lds_ptr*)(buf + (4 * i + wave) * 1024), 16, int(a_off[i]), ko, 0, 0);
      __builtin_amdgcn_raw_ptr_buffer_load_lds(w_rsrc, (lds_ptr*)(buf + L_TILE_BYTES + (4 * i + wave) * 1024), 16, int(w_off[i]), ko, 0, 0);
    }
  };
  f32x4 acc[4][4];
#pragma unroll
  for (int mb = 0; mb < 4; ++mb)
#pragma unroll
    for (int nb = 0; nb < 4; ++nb) acc[mb][nb] = f32x4{0.f, 0.f, 0.f, 0.f};

  const int a_read = (wm * 64 + lr) * 64 + ((lq ^ (lr >> 2)) * 16), w_read = L_TILE_BYTES + (wn * 64 + lr) * 64 + ((lq ^ (lr >> 2)) * 16);
  auto compute = [&](const uint8_t* buf) {
    bf16x8 af[4];
    u32x4 wf[4];
#pragma unroll
    for (int b = 0; b < 4; ++b) {
      af[b] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const u32x4*>(buf + a_read + b * 16 * 64));
      wf[b] = *reinterpret_cast<const u32x4*>(buf + w_read + b * 16 * 64);
    }
    // the weights are the FIRST operand: the result block is C^T, a lane then holds four neighbouring columns of one row
#pragma unroll
    for (int mb = 0; mb < 4; ++mb)
#pragma unroll
      for (int nb = 0; nb < 4; ++nb) acc[mb][nb] = mfma_bf16(wf[nb], af[mb], acc[mb][nb]);
  };
  auto step = [&](int kt, const uint8_t* cur, uint8_t* next) {
    fetch(next, kt + 1);                                     // last read a step ago, before the barrier
    __builtin_amdgcn_sched_barrier(0);
    compute(cur);
    __builtin_amdgcn_sched_barrier(0);
    __syncthreads();                                         // waits for the requests above as well
  };
  int kt = kt0;
  if constexpr (NB == 2) {
    fetch(buf0, kt0);
    __syncthreads();
#pragma unroll 1
    for (; kt + 2 <= kt1; kt += 2) {
      step(kt, buf0, buf1);
      step(kt + 1, buf1, buf0);
    }
    if (kt < kt1) compute(buf0);
  } else {
    __shared__ __align__(1024) uint8_t buf2[2 * L_TILE_BYTES], buf3[2 * L_TILE_BYTES];
    auto deep = [&](int t, const uint8_t* cur, uint8_t* next) {
      __builtin_amdgcn_s_waitcnt(8 | (7 << 4) | (15 << 8));  // all but the eight requests of tiles t + 1 and t + 2: tile t is there
      asm volatile("" ::: "memory");
      __builtin_amdgcn_s_barrier();
      asm volatile("" ::: "memory");
      __builtin_amdgcn_sched_barrier(0);
      fetch(next, t + 3);                                    // last read a step ago, before the barrier
      __builtin_amdgcn_sched_barrier(0);
      compute(cur);
      __builtin_amdgcn_sched_barrier(0);
    };
    fetch(buf0, kt0);
    fetch(buf1, kt0 + 1);
    fetch(buf2, kt0 + 2);
#pragma unroll 1
    for (; kt + 4 <= kt1; kt += 4) {
      deep(kt, buf0, buf3);
      deep(kt + 1, buf1, buf0);
      deep(kt + 2, buf2, buf1);
      deep(kt + 3, buf3, buf2);
    }
    __syncthreads();                                         // waits for every request: up to three tiles are left, and none is in flight
    if (kt < kt1) compute(buf0);
    if (kt + 1 < kt1) compute(buf1);
    if (kt + 2 < kt1) compute(buf2);
  }
  // ---- epilogue: lane (lr, lq) holds row wm*64 + mb*16 + lr, columns wn*64 + nb*16 + 4 lq .. + 3.  Stored from there an access touches 64 (32 in
  // bf16) bytes of each of 16 rows; 32 rows at a time go through LDS (units of 16 bytes XOR-swizzled by the row, each wave in
  // 8 KB of its own), so that 16 lanes move a whole row of the wave's 64 columns.
  __syncthreads();
  float* stage = reinterpret_cast<float*>((wave < 2 ? buf0 : buf1) + (wave & 1) * L_TILE_BYTES);
  const int col = n0 + wn * 64 + lr * 4;
  f32x4 bias = {0.f, 0.f, 0.f, 0.f};
  if (la.ksplit == 1 && la.bias) bias = *reinterpret_cast<const f32x4*>(la.bias + col);
#pragma unroll
  for (int h = 0; h < 2; ++h) {
#pragma unroll
    for (int m2 = 0; m2 < 2; ++m2)
#pragma unroll
      for (int nb = 0; nb < 4; ++nb) *reinterpret_cast<f32x4*>(stage + (m2 * 16 + lr) * 64 + ((nb * 4 + lq) ^ lr) * 4) = acc[h * 2 + m2][nb];
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const int r = i * 4 + lq, row = m0 + wm * 64 + h * 32 + r;
      f32x4 v = *reinterpret_cast<const f32x4*>(stage + r * 64 + (lr ^ (r & 15)) * 4);
      if (row >= la.M) continue;
      const size_t o = size_t(row) * la.n + col;
      if (la.ksplit > 1) {
        *reinterpret_cast<f32x4*>(la.part + size_t(blockIdx.z) * la.M * la.n + o) = v;
        continue;
      }
      v = v + bias;
      if (la.residual) v = v + *reinterpret_cast<const f32x4*>(la.residual + o);
      if (la.relu) { v.x = fmaxf(v.x, 0.f); v.y = fmaxf(v.y, 0.f); v.z = fmaxf(v.z, 0.f); v.w = fmaxf(v.w, 0.f); }
      if (la.c32) *reinterpret_cast<f32x4*>(la.c32 + o) = v;
      if (la.c16) {
        uint2 q;
        q.x = pack_bf16x2(v.x, v.y);
        q.y = pack_bf16x2(v.z, v.w);
        *reinterpret_cast<uint2*>(la.c16 + o) = q;
      }
    }
  }
}

// Split launches: C = (sum over the k-shares, in order) + bias [+ residual] [ReLU]; four columns per thread.
__global__ __launch_bounds__(256) void k_lin_finish(const LinArgs la) {
  const size_t i = (size_t(blockIdx.x) * 256 + threadIdx.x) * 4, total = size_t(la.M) * la.n;
  if (i >= total) return;
  float4 v = *reinterpret_cast<const float4*>(la.part + i);
  for (int z = 1; z < la.ksplit; ++z) {
    const float4 t = *reinterpret_cast<const float4*>(la.part + size_t(z) * total + i);
    v.x += t.x; v.y += t.y; v.z += t.z; v.w += t.w;
  }
  const int col = int(i % size_t(la.n));
  if (la.bias) { const float4 t = *reinterpret_cast<const float4*>(la.bias + col); v.x += t.x; v.y += t.y; v.z += t.z; v.w += t.w; }
  if (la.residual) { const float4 t = *reinterpret_cast<const float4*>(la.residual + i); v.x += t.x; v.y += t.y; v.z += t.z; v.w += t.w; }
  if (la.relu) { v.x = fmaxf(v.x, 0.f); v.y = fmaxf(v.y, 0.f); v.z = fmaxf(v.z, 0.f); v.w = fmaxf(v.w, 0.f); }
  if (la.c32) *reinterpret_cast<float4*>(la.c32 + i) = v;
  if (la.c16) {
    uint2 o;
    o.x = pack_bf16x2(v.x, v.y);
    o.y = pack_bf16x2(v.z, v.w);
    *reinterpret_cast<uint2*>(la.c16 + i) = o;
  }
}

// ---- attention -----------------------------------------------------------------------------------------------
// qkv: fp32 [S*T, 3*dm] (queries, keys, values); out: bf16 [S*T, dm].  A work-group takes 16 NW queries of one head (a wave 16 of them) and
// streams the keys in tiles of 32 through LDS.
// Products are fp32 products on the bf16 matrix cores: every operand (queries, keys, values, probabilities) is cut into three bf16 pieces
// that add up to it exactly, and the six largest of their nine products are summed in fp32; what is left out is at most the rounding of ONE
// fp32 product, with either sign (bf16_pieces.h).  Six 16x16x32 operations take 96 cycles where the fp32 matrix cores take 256, and the
// pieces of keys and values are made once per work-group, on their way into LDS.  (fp32 matrix cores: 157 us on 128 sequences of 256
// tokens, 6 heads of 64.)
// Scores are computed TRANSPOSED (keys x queries), so that a lane's eight accumulator values are eight keys of ITS query (lane % 16): the
// softmax of a query then needs its own lane's values and those of the three lanes 16, 32, 48 further on, and the probabilities
// already sit where the second product wants them: k-slot 8 lq + 4 b + r of it is key 16 b + 4 lq + r, the order the values are stored in.
// 128 sequences of 256 tokens, 6 heads of 64: 80 us, matrix cores busy 40 % of the time (90 with loads at 64-bit addresses and sums and maxima through
// LDS); 16 of 1024 tokens, the whole router 453 -> 424.  32 queries a wave, which halve the reads of LDS, were no faster (81 us, 16 x 1024 460).
constexpr int ATT_KEYS = 32;

// Eight values as three operands of eight bf16.
static __device__ __forceinline__ void cut3x8(const float (&v)[8], u32x4 (&o)[3]) {
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    uint32_t p1, p2, p3;
    cut3_pair(v[2 * i], v[2 * i + 1], p1, p2, p3);
    o[0][i] = p1; o[1][i] = p2; o[2][i] = p3;
  }
}
static __device__ __forceinline__ f32x4 mfma_cut3(const u32x4 (&a)[3], const u32x4 (&b)[3], f32x4 c) {
  const bf16x8 b0 = __builtin_bit_cast(bf16x8, b[0]), b1 = __builtin_bit_cast(bf16x8, b[1]), b2 = __builtin_bit_cast(bf16x8, b[2]);
  c = mfma_bf16(a[2], b0, c);               // small terms first
  c = mfma_bf16(a[0], b2, c);
  c = mfma_bf16(a[1], b1, c);
  c = mfma_bf16(a[1], b0, c);
  c = mfma_bf16(a[0], b1, c);
  return mfma_bf16(a[0], b0, c);
}

// A wave's 16 queries q0 .. q0 + 15 against all keys on the fp32 matrix cores, operands straight from memory: 16 keys at a time, lane group lq
// takes the quarter lq of the dimensions and the keys 4 lq .. 4 lq + 3.  base: the sample's rows at the head's first column.
template <int DH>
static __device__ __forceinline__ void attend_fp32(const float* __restrict__ base, size_t ld, int dm, int T, float scale, int q0,
                                                   f32x4 (&o)[DH / 16], float& l_run) {
  constexpr int QS = DH / 4, CB = DH / 16;
  const int lane = threadIdx.x & 63, lr = lane & 15, lq = lane >> 4;
  const float* qp = base + size_t(min(q0 + lr, T - 1)) * ld + lq * QS;
  float qf[QS], m_run = -INFINITY;
  l_run = 0.f;
#pragma unroll
  for (int i = 0; i < QS; i += 4) {
    const float4 v = *reinterpret_cast<const float4*>(qp + i);
    qf[i] = v.x * scale; qf[i + 1] = v.y * scale; qf[i + 2] = v.z * scale; qf[i + 3] = v.w * scale;
  }
#pragma unroll
  for (int cb = 0; cb < CB; ++cb) o[cb] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll 1
  for (int k0 = 0; k0 < T; k0 += 16) {
    float kf[QS], vf[4][CB];                                 // rows past T repeat row T - 1
    const float* kp = base + dm + size_t(min(k0 + lr, T - 1)) * ld + lq * QS;
#pragma unroll
    for (int i = 0; i < QS; i += 4) {
      const float4 v = *reinterpret_cast<const float4*>(kp + i);
      kf[i] = v.x; kf[i + 1] = v.y; kf[i + 2] = v.z; kf[i + 3] = v.w;
    }
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const float* vp = base + 2 * dm + size_t(min(k0 + 4 * lq + r, T - 1)) * ld + lr;
#pragma unroll
      for (int cb = 0; cb < CB; ++cb) vf[r][cb] = vp[cb * 16];
    }
    f32x4 sc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int i = 0; i < QS; ++i) sc = __builtin_amdgcn_mfma_f32_16x16x4f32(kf[i], qf[i], sc, 0, 0, 0);
    // lane (lr, lq) holds the scores of query q0 + lr against keys k0 + 4 lq + r
    float p[4], tmax = -INFINITY;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      p[r] = k0 + 4 * lq + r < T ? sc[r] : -INFINITY;
      tmax = fmaxf(tmax, p[r]);
    }
    tmax = fmaxf(tmax, __shfl_xor(tmax, 16));
    tmax = fmaxf(tmax, __shfl_xor(tmax, 32));
    const float m_new = fmaxf(m_run, tmax);
    const float alpha = __expf(m_run - m_new);               // exp(-inf) = 0 on the first tile
    float tsum = 0.f;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      p[r] = __expf(p[r] - m_new);
      tsum += p[r];
    }
    tsum += __shfl_xor(tsum, 16);
    tsum += __shfl_xor(tsum, 32);
    l_run = l_run * alpha + tsum;
    m_run = m_new;
#pragma unroll
    for (int cb = 0; cb < CB; ++cb)
#pragma unroll
      for (int r = 0; r < 4; ++r) o[cb][r] *= alpha;
#pragma unroll
    for (int r = 0; r < 4; ++r)                              // dead keys have p = 0
#pragma unroll
      for (int cb = 0; cb < CB; ++cb) o[cb] = __builtin_amdgcn_mfma_f32_16x16x4f32(vf[r][cb], p[r], o[cb], 0, 0, 0);
  }
}

// lane (lr, lq) holds out[q0 + lr][16 cb + 4 lq + r], not yet divided by the sum of the weights
template <int DH>
static __device__ __forceinline__ void store_queries(const f32x4 (&o)[DH / 16], float l_run, uint16_t* __restrict__ out, int s, int T, int dm,
                                                     int head, int q0) {
  const int lane = threadIdx.x & 63, lr = lane & 15, lq = lane >> 4;
  if (q0 + lr >= T) return;
  const float inv = 1.f / l_run;
  uint16_t* op = out + (size_t(s) * T + q0 + lr) * dm + head * DH + 4 * lq;
#pragma unroll
  for (int cb = 0; cb < DH / 16; ++cb) {
    uint2 v;
    v.x = pack_bf16x2(o[cb][0] * inv, o[cb][1] * inv);
    v.y = pack_bf16x2(o[cb][2] * inv, o[cb][3] * inv);
    *reinterpret_cast<uint2*>(op + cb * 16) = v;
  }
}

// Samples of a few tokens: a wave per 16 queries, all of the sample in one work-group.
template <int DH>
__global__ __launch_bounds__(256) void k_attention_fp32(const float* __restrict__ qkv, uint16_t* __restrict__ out, int S, int T, int dm,
                                                         float scale) {
  const int q0 = int(threadIdx.x >> 6) * 16, head = blockIdx.y, s = blockIdx.z;
  const size_t ld = size_t(3) * dm;
  f32x4 o[DH / 16];
  float l_run;
  attend_fp32<DH>(qkv + size_t(s) * T * ld + head * DH, ld, dm, T, scale, q0, o, l_run);
  store_queries<DH>(o, l_run, out, s, T, dm, head, q0);
}

// f over the four lanes of a query (16 apart), in each of them: exchanges of rows of 16 lanes, no LDS.
template <typename F> static __device__ __forceinline__ float of_four(float v, F f) {
  const auto a = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  v = f(__uint_as_float(a[0]), __uint_as_float(a[1]));
  const auto b = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return f(__uint_as_float(b[0]), __uint_as_float(b[1]));
}

// NBUF: key tiles in LDS, one being read and, with two, the next one being stored
template <int DH, int NW, int NBUF>
__global__ __launch_bounds__(NW * 64) void k_attention(const float* __restrict__ qkv, uint16_t* __restrict__ out, int S, int T, int dm,
                                                        float scale) {
  constexpr int KD = DH < 32 ? 32 : DH;           // dimensions as the matrix cores see them (heads of 16: the upper half is zero)
  constexpr int JS = KD / 32, CB = DH / 16;
  constexpr int K_ROW = KD * 2 + 16;              // LDS bytes of a key's pieces; the pad spreads 16 rows over the banks
  constexpr int V_ROW = ATT_KEYS * 2 + 16;        // ... of a dimension's 32 keys
  constexpr int K_PLANE = ATT_KEYS * K_ROW, V_PLANE = DH * V_ROW;
  constexpr int NT = NW * 64, TASKS = 8 * DH, ITERS = (TASKS + NT - 1) / NT;
  __shared__ __align__(16) uint8_t kl[NBUF][3 * K_PLANE];
  __shared__ __align__(16) uint8_t vl[NBUF][3 * V_PLANE];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int lr = lane & 15, lq = lane >> 4;
  const int q0 = (blockIdx.x * NW + wave) * 16;
  const int head = blockIdx.y, s = blockIdx.z;
  const size_t ld = size_t(3) * dm;
  const float* base = qkv + size_t(s) * T * ld + head * DH;
  if constexpr (KD > DH) {                        // the zero half of the keys, every buffer, written once
    for (int i = tid; i < NBUF * 3 * ATT_KEYS; i += NT) {
      uint8_t* row = kl[i / (3 * ATT_KEYS)] + (i % (3 * ATT_KEYS)) * K_ROW + DH * 2;
      *reinterpret_cast<u32x4*>(row) = u32x4{0u, 0u, 0u, 0u};
      *reinterpret_cast<u32x4*>(row + 16) = u32x4{0u, 0u, 0u, 0u};
    }
  }
  // staging: the first 4 DH tasks take eight dimensions of a key, the others eight keys of a dimension; keys past T read as zeros, past the end of the
  // tile's buffer descriptor (as 64-bit addresses of clamped rows the ten loads of a task cost 27 quarter-rate multiplications)
  float st[ITERS][8];
  const uint32_t pitch = uint32_t(ld) * 4u;
  uint32_t at[ITERS];                             // byte offset of a task's first value behind the tile's first row
  bool is_key[ITERS];
#pragma unroll
  for (int it = 0; it < ITERS; ++it) {
    const int id = tid + it * NT;
    is_key[it] = id < 4 * DH;
    at[it] = is_key[it] ? uint32_t(id / (DH / 8)) * pitch + uint32_t(dm + (id % (DH / 8)) * 8) * 4u
                        : uint32_t(4 * ((id - 4 * DH) / DH)) * pitch + uint32_t(2 * dm + (id - 4 * DH) % DH) * 4u;
  }
  auto load_tile = [&](int k0) {
    const buf_rsrc rows = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(base + size_t(k0) * ld), 0, uint32_t(min(ATT_KEYS, T - k0)) * pitch - uint32_t(head * DH) * 4u,
                                                            0x00020000);
#pragma unroll
    for (int it = 0; it < ITERS; ++it) {
      if (is_key[it]) {
        const u32x4 x = buf_load128(rows, int(at[it]), 0), y = buf_load128(rows, int(at[it]) + 16, 0);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          st[it][i] = __uint_as_float(x[i]);
          st[it][4 + i] = __uint_as_float(y[i]);
        }
      } else if (tid + it * NT < TASKS) {
#pragma unroll
        for (int i = 0; i < 8; ++i) st[it][i] = __uint_as_float(buf_load32(rows, int(at[it] + uint32_t((i >> 2) * 16 + (i & 3)) * pitch), 0));
      }
    }
  };
  auto store_tile = [&](int buf) {
#pragma unroll
    for (int it = 0; it < ITERS; ++it) {
      const int id = tid + it * NT;
      if (id < TASKS) {
        u32x4 o[3];
        cut3x8(st[it], o);
        const bool key = id < 4 * DH;
        uint8_t* p = key ? kl[buf] + (id / (DH / 8)) * K_ROW + (id % (DH / 8)) * 16
                         : vl[buf] + ((id - 4 * DH) % DH) * V_ROW + ((id - 4 * DH) / DH) * 16;
        const int plane = key ? K_PLANE : V_PLANE;
#pragma unroll
        for (int i = 0; i < 3; ++i) *reinterpret_cast<u32x4*>(p + i * plane) = o[i];
      }
    }
  };
  load_tile(0);
  // queries, scaled: lane (lr, lq) holds dimensions 32 j + 8 lq .. + 7 of query q0 + lr
  u32x4 qf[JS][3];
  {
    const float* qp = base + size_t(min(q0 + lr, T - 1)) * ld;
#pragma unroll
    for (int j = 0; j < JS; ++j) {
      float v[8];
      const int d = 32 * j + 8 * lq;
#pragma unroll
      for (int i = 0; i < 8; i += 4) {
        const float4 x = d < DH ? *reinterpret_cast<const float4*>(qp + d + i) : make_float4(0.f, 0.f, 0.f, 0.f);
        v[i] = x.x * scale; v[i + 1] = x.y * scale; v[i + 2] = x.z * scale; v[i + 3] = x.w * scale;
      }
      cut3x8(v, qf[j]);
    }
  }
  f32x4 o[CB];
  float m_run = -INFINITY, l_run = 0.f;
#pragma unroll
  for (int cb = 0; cb < CB; ++cb) o[cb] = f32x4{0.f, 0.f, 0.f, 0.f};
  store_tile(0);
  __syncthreads();
  int buf = 0;
  for (int k0 = 0; k0 < T; k0 += ATT_KEYS, buf ^= NBUF - 1) {
    const bool more = NW > 2 && k0 + ATT_KEYS < T;          // uniform over the work-group; two waves have one tile of keys
    if (more) load_tile(k0 + ATT_KEYS);
    if (q0 < T) {                                           // uniform over the wave: it has queries
      // ---- scores^T[key][query]
      __builtin_amdgcn_s_setprio(1);                        // products ahead of other waves' softmax and staging
      f32x4 sc[2];
#pragma unroll
      for (int kb = 0; kb < 2; ++kb) {
        sc[kb] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int j = 0; j < JS; ++j) {
          u32x4 kf[3];
#pragma unroll
          for (int i = 0; i < 3; ++i)
            kf[i] = *reinterpret_cast<const u32x4*>(kl[buf] + i * K_PLANE + (kb * 16 + lr) * K_ROW + j * 64 + lq * 16);
          sc[kb] = mfma_cut3(kf, qf[j], sc[kb]);
        }
      }
      __builtin_amdgcn_sched_barrier(0);
      __builtin_amdgcn_s_setprio(0);
      // lane (lr, lq) holds the scores of query q0 + lr against keys k0 + 16 kb + 4 lq + r
      float p[8], tmax = -INFINITY;
#pragma unroll
      for (int i = 0; i < 8; ++i) p[i] = sc[i >> 2][i & 3];
      if (k0 + ATT_KEYS > T) {                              // uniform: the last tile may have keys past T
#pragma unroll
        for (int i = 0; i < 8; ++i) p[i] = k0 + (i >> 2) * 16 + 4 * lq + (i & 3) < T ? p[i] : -INFINITY;
      }
#pragma unroll
      for (int i = 0; i < 8; ++i) tmax = fmaxf(tmax, p[i]);
      const float m_new = fmaxf(m_run, of_four(tmax, [](float a, float b) { return fmaxf(a, b); }));     // finite: key k0 itself is live
      const float alpha = __expf(m_run - m_new);            // exp(-inf) = 0 on the first tile
      float tsum = 0.f;
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        p[i] = __expf(p[i] - m_new);
        tsum += p[i];
      }
      l_run = l_run * alpha + tsum;                         // of the lane's own keys; the four lanes of a query share m_run
      m_run = m_new;
      u32x4 pf[3];
      cut3x8(p, pf);                                        // dead keys have p = 0
      // ---- out^T[c][query] += V^T P^T
      __builtin_amdgcn_sched_barrier(0);
      __builtin_amdgcn_s_setprio(1);
#pragma unroll
      for (int cb = 0; cb < CB; ++cb) {
#pragma unroll
        for (int r = 0; r < 4; ++r) o[cb][r] *= alpha;
        u32x4 vf[3];
#pragma unroll
        for (int i = 0; i < 3; ++i) vf[i] = *reinterpret_cast<const u32x4*>(vl[buf] + i * V_PLANE + (cb * 16 + lr) * V_ROW + lq * 16);
        o[cb] = mfma_cut3(vf, pf, o[cb]);
      }
      __builtin_amdgcn_sched_barrier(0);
      __builtin_amdgcn_s_setprio(0);
    }
    if constexpr (NBUF == 2) {
      if (more) store_tile(buf ^ 1);                        // last read a tile ago, before the barrier below
      __syncthreads();
    } else if (more) {
      __syncthreads();                                      // the tile has been read
      store_tile(0);
      __syncthreads();
    }
  }
  // An infinite operand, or one whose first piece rounds to infinity, leaves NaN or infinite rests, and NaN results where the product itself
  // has a value (a key whose score is minus infinity has weight 0).  Every such piece reaches the sum of the weights or an output of the
  // query, so a wave whose results are not all finite takes them again from whole operands.
  l_run = of_four(l_run, [](float a, float b) { return a + b; });
  float check = l_run * 0.f;
#pragma unroll
  for (int cb = 0; cb < CB; ++cb)
#pragma unroll
    for (int r = 0; r < 4; ++r) check = fmaf(o[cb][r], 0.f, check);
  if (__ballot(check != check) != 0ull) attend_fp32<DH>(base, ld, dm, T, scale, q0, o, l_run);
  store_queries<DH>(o, l_run, out, s, T, dm, head, q0);
}

// ---- LayerNorm -----------------------------------------------------------------------------------------------
static __device__ __forceinline__ float wave_sum_f(float v) {
#pragma unroll
  for (int d = 32; d >= 1; d >>= 1) v += __shfl_xor(v, d);
  return v;
}

constexpr int LN_MAX_PER_LANE = 32;      // rows of up to 2048 elements
__global__ __launch_bounds__(256) void k_layer_norm(const float* __restrict__ x, const float* __restrict__ g, const float* __restrict__ b,
                                                     int M, int n, float* __restrict__ y32, uint16_t* __restrict__ y16) {
  const int row = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
  if (row >= M) return;
  const float* xr = x + size_t(row) * n;
  float v[LN_MAX_PER_LANE];
  float sum = 0.f;
#pragma unroll
  for (int i = 0; i < LN_MAX_PER_LANE; ++i) {
    const int c = lane + 64 * i;
    v[i] = c < n ? xr[c] : 0.f;
    sum += v[i];
  }
  const float mu = wave_sum_f(sum) / float(n);
  float sq = 0.f;
#pragma unroll
  for (int i = 0; i < LN_MAX_PER_LANE; ++i) {
    const int c = lane + 64 * i;
    const float d = c < n ? v[i] - mu : 0.f;
    sq += d * d;
  }
  const float rstd = 1.0f / sqrtf(wave_sum_f(sq) / float(n) + 1e-5f);
#pragma unroll
  for (int i = 0; i < LN_MAX_PER_LANE; ++i) {
    const int c = lane + 64 * i;
    if (c < n) {
      const float r = (v[i] - mu) * rstd * g[c] + b[c];
      if (y32) y32[size_t(row) * n + c] = r;
      if (y16) y16[size_t(row) * n + c] = float_to_bf16_rne(r);
    }
  }
}

// The last LayerNorm and the mean over a sample's tokens in one pass: a work-group takes one chunk of a sample's rows, wave w the rows
// w, w + NW, ... of it; every lane adds its columns of the normalized rows in order, the waves' sums are added in wave order.
// part[s][chunk][n] holds the chunk's sum, or with a single chunk the mean itself.  (Two kernels with the normalized rows written and
// read in between took 25 + 12 us on 32768 rows of 384; this and k_pool_f32 11 + 5.)  PL: columns per lane, the smallest of 8, 16 and 32 that holds the
// width, with 16, 8 or 4 waves: 32 samples of 33 tokens of 1024 8.6 us, with the widest 16.3 (two kernels 13.1); of 2048 19.8 (23.0).
template <int PL, int NW>
__global__ __launch_bounds__(NW * 64) void k_ln_pool(const float* __restrict__ x, const float* __restrict__ g, const float* __restrict__ b, int T,
                                                      int n, int chunk_rows, float* __restrict__ part) {
  __shared__ float red[NW][PL * 64];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int s = blockIdx.y, c0 = blockIdx.x * chunk_rows, c1 = min(T, c0 + chunk_rows);
  float acc[PL], gl[PL], bl[PL];
#pragma unroll
  for (int i = 0; i < PL; ++i) {
    const int c = lane + 64 * i;
    acc[i] = 0.f;
    gl[i] = c < n ? g[c] : 0.f;
    bl[i] = c < n ? b[c] : 0.f;
  }
  for (int t = c0 + wave; t < c1; t += NW) {
    const float* xr = x + (size_t(s) * T + t) * n;
    float v[PL], sum = 0.f, sq = 0.f;
#pragma unroll
    for (int i = 0; i < PL; ++i) {
      const int c = lane + 64 * i;
      v[i] = c < n ? xr[c] : 0.f;
      sum += v[i];
    }
    const float mu = wave_sum_f(sum) / float(n);
#pragma unroll
    for (int i = 0; i < PL; ++i) {
      const float d = lane + 64 * i < n ? v[i] - mu : 0.f;
      sq += d * d;
    }
    const float rstd = 1.0f / sqrtf(wave_sum_f(sq) / float(n) + 1e-5f);
#pragma unroll
    for (int i = 0; i < PL; ++i) acc[i] += (v[i] - mu) * rstd * gl[i] + bl[i];       // columns past n: never read again
  }
#pragma unroll
  for (int i = 0; i < PL; ++i) red[wave][lane + 64 * i] = acc[i];
  __syncthreads();
  for (int c = threadIdx.x; c < n; c += NW * 64) {
    float v = red[0][c];
#pragma unroll
    for (int w = 1; w < NW; ++w) v += red[w][c];
    part[(size_t(s) * gridDim.x + blockIdx.x) * n + c] = gridDim.x == 1 ? __fdiv_rn(v, float(T)) : v;
  }
}

// pooled[s][c] = (sum over the chunks of part[s][.][c], in order) / T
__global__ __launch_bounds__(256) void k_pool_f32(const float* __restrict__ part, float* __restrict__ pooled, int S, int chunks, int n, int T) {
  const size_t i = size_t(blockIdx.x) * 256 + threadIdx.x;
  if (i >= size_t(S) * n) return;
  const float* p = part + (i / n) * size_t(chunks) * n + i % n;
  float v = p[0];
  for (int c = 1; c < chunks; ++c) v += p[size_t(c) * n];
  pooled[i] = __fdiv_rn(v, float(T));
}

// ---- host side -------------------------------------------------------------------------------------------------
namespace {
constexpr int LIN_SPLIT_MAX = 16;            // most k-shares of one product
constexpr int LIN_SPLIT_MAX_ROWS = 512;      // products with more rows fill the chip without splitting

struct NlpLayout {
  size_t w_in, wqkv1, wo1, wff1, wff2, wqkv2, wo2;          // bf16 parameter copies
  size_t t32a, t32b, t32c, t16a, t16b, qkv, hid, part, pooled, head, total;
};

NlpLayout nlp_layout(int S, int T, const moqe_nlp_router& r) {
  NlpLayout L;
  const size_t M = size_t(S) * T, dm = r.dm;
  size_t o = 0;
  auto take = [&](size_t bytes) { const size_t at = o; o += align256(bytes); return at; };
  L.w_in = take(dm * r.d * 2);
  L.wqkv1 = take(3 * dm * dm * 2);
  L.wo1 = take(dm * dm * 2);
  L.wff1 = take(size_t(r.d_ff) * dm * 2);
  L.wff2 = take(size_t(r.d_ff) * dm * 2);
  L.wqkv2 = take(3 * dm * dm * 2);
  L.wo2 = take(dm * dm * 2);
  L.t32a = take(M * dm * 4);
  L.t32b = take(M * dm * 4);
  L.t32c = take(M * dm * 4);
  L.t16a = take(M * dm * 2);
  L.t16b = take(M * dm * 2);
  L.qkv = take(M * 3 * dm * 4);
  L.hid = take(M * size_t(r.d_ff) * 2);
  const size_t widest = std::max<size_t>(3 * dm, size_t(r.d_ff));
  L.part = take(M <= size_t(LIN_SPLIT_MAX_ROWS) ? size_t(LIN_SPLIT_MAX) * M * widest * 4 : 0);   // k-shares of launches with few rows
  L.pooled = take(size_t(S) * dm * 4);
  L.head = take(route_ws_bytes(S, 1, r.head));
  L.total = o;
  return L;
}

// Tiles of the same rows go to the same XCD from eight row tiles on; fewer would leave XCDs idle (64 x 1 tokens, one row tile, all its
// work-groups on one XCD: the router 105 us, spread 102; with eight as the line 3072 rows take 159 us, with 64 164).  What does not make
// a whole group of eight is spread too: 18 row tiles (width 2048) 578 us, dealt as a third group that only two XCDs share 636.
constexpr int LIN_XCD_ROWS = 8;
// A launch that gives a CU at most one work-group has nothing to hide a k-tile's way from memory behind but the tiles after it: it keeps
// three in flight (four buffers).  The router at 1000 rows 195 -> 171 us, 1536 rows 187 -> 169, 6144 rows 227 -> 209; with up to
// two work-groups to a CU on this path 6144 rows take 213 and 12000 rows 327 instead of 320.
constexpr unsigned LIN_DEEP_MAX = 256;

int32_t lin(const uint16_t* a, const uint16_t* w, const float* bias, const float* residual, float* c32, uint16_t* c16, int M, int n,
            int k, bool relu, float* part, hipStream_t st) {
  LinArgs la{a, w, bias, residual, c32, c16, M, n, k, relu ? 1 : 0, 0, 1, part};
  const int m_tiles = (M + LBM - 1) / LBM, wgs = (n / LBN) * m_tiles;
  // few rows: the k-tiles are shared out over more work-groups (at least 128 values of k each), summed by a second launch
  if (M <= LIN_SPLIT_MAX_ROWS)
    while (wgs * la.ksplit < 96 && la.ksplit * 256 <= k && la.ksplit < LIN_SPLIT_MAX) la.ksplit *= 2;
  la.by_xcd = m_tiles >= LIN_XCD_ROWS;
  ProfileScope ps(MOQE_PK_ROUTE, st);
  const dim3 g(unsigned(wgs), 1, la.ksplit);
  if (g.x * g.z <= LIN_DEEP_MAX) hipLaunchKernelGGL(k_lin<4>, g, dim3(256), 0, st, la);
  else hipLaunchKernelGGL(k_lin<2>, g, dim3(256), 0, st, la);
  if (la.ksplit > 1)
    hipLaunchKernelGGL(k_lin_finish, dim3(unsigned((size_t(M) * n / 4 + 255) / 256)), dim3(256), 0, st, la);
  return check_launch("route_nlp(linear)");
}

template <int DH>
void launch_attention(const float* qkv, uint16_t* out, int S, int T, int dm, int heads, float scale, hipStream_t st) {
  // A sample of at most 16 tokens is ONE tile of the fp32 matrix cores: nothing is staged, nothing shared (384 samples of one token, 8 heads
  // of 128: 8.2 us against 33.5; 24 heads of 16: 6.2 against 12.5).  With heads of 16, where half of a bf16 operation is padding, up to 48 (128
  // samples of 48: 13.5 against 16.0; of 64: 18.6 against 17.4).  Longer ones share the cut keys among waves: two up to
  // 32 tokens, one tile of keys (128 x 17, heads of 32: 5.5 against 6.3 with four; of 128, 14.8 against 15.8 but 19.3 against 18.0 at 32), then four, and eight from 65
  // tokens on (128 x 65, heads of 64: 16.9 against 23.8) but for 129 to 192, which are three work-groups of four and would be two half-filled
  // ones of eight (64 x 129, heads of 16: 41 against 55; of 128: 148 against 177; of 64: 28.7 against 26.9).
  // One key buffer, so that two to five work-groups share a CU (128 x 33, heads of 128: 48 us, with two buffers 74); eight waves of heads of 128 fill a CU's
  // registers by themselves and take two (16 x 512: 236 against 257).
  if (T <= (DH == 16 ? 48 : 16))
    hipLaunchKernelGGL(k_attention_fp32<DH>, dim3(1, heads, S), dim3((T + 15) / 16 * 64), 0, st, qkv, out, S, T, dm, scale);
  else if (T <= ATT_KEYS && DH <= 64)
    hipLaunchKernelGGL((k_attention<DH <= 64 ? DH : 64, 2, 1>), dim3(1, heads, S), dim3(128), 0, st, qkv, out, S, T, dm, scale);
  else if (T <= 64 || (T > 128 && T <= 192))
    hipLaunchKernelGGL((k_attention<DH, 4, 1>), dim3((T + 63) / 64, heads, S), dim3(256), 0, st, qkv, out, S, T, dm, scale);
  else
    hipLaunchKernelGGL((k_attention<DH, 8, DH == 128 ? 2 : 1>), dim3((T + 127) / 128, heads, S), dim3(512), 0, st, qkv, out, S, T, dm, scale);
}

int32_t layer_norm(const float* x, const float* g, const float* b, int M, int n, float* y32, uint16_t* y16, hipStream_t st) {
  ProfileScope ps(MOQE_PK_ROUTE, st);
  hipLaunchKernelGGL(k_layer_norm, dim3((M + 3) / 4), dim3(256), 0, st, x, g, b, M, n, y32, y16);
  return check_launch("route_nlp(layer norm)");
}
}  // namespace

int32_t launch_nlp_attention(const float* qkv, uint16_t* out, int S, int T, int dm, int heads, hipStream_t st) {
  const int dh = dm / heads;
  const float scale = 1.0f / sqrtf(float(dh));
  ProfileScope ps(MOQE_PK_ROUTE, st);
  switch (dh) {
    case 16:  launch_attention<16>(qkv, out, S, T, dm, heads, scale, st); break;
    case 32:  launch_attention<32>(qkv, out, S, T, dm, heads, scale, st); break;
    case 64:  launch_attention<64>(qkv, out, S, T, dm, heads, scale, st); break;
    default:  launch_attention<128>(qkv, out, S, T, dm, heads, scale, st); break;
  }
  return check_launch("route_nlp(attention)");
}

int32_t check_nlp_router(const moqe_nlp_router* r, const char* who) {
  if (!r) return set_error(MOQE_E_NULL, "%s: router is NULL", who);
  const void* need[] = {r->w_in, r->b_in, r->wqkv1, r->bqkv1, r->wo1, r->bo1, r->ln1_g, r->ln1_b, r->w_ff1, r->b_ff1, r->w_ff2,
                        r->b_ff2, r->ln2_g, r->ln2_b, r->wqkv2, r->bqkv2, r->wo2, r->bo2, r->ln3_g, r->ln3_b};
  for (const void* p : need)
    if (!p) return set_error(MOQE_E_NULL, "%s: a parameter pointer is NULL", who);
  const void* mats[] = {r->w_in, r->wqkv1, r->wo1, r->w_ff1, r->w_ff2, r->wqkv2, r->wo2};
  for (const void* p : mats)
    if (reinterpret_cast<uintptr_t>(p) % 16) return set_error(MOQE_E_SHAPE, "%s: parameter matrices must be 16-byte aligned", who);
  const void* vecs[] = {r->b_in, r->bqkv1, r->bo1, r->b_ff1, r->b_ff2, r->bqkv2, r->bo2};
  for (const void* p : vecs)
    if (reinterpret_cast<uintptr_t>(p) % 16) return set_error(MOQE_E_SHAPE, "%s: bias vectors must be 16-byte aligned", who);
  if (r->d <= 0 || r->d % 64 || r->dm <= 0 || r->dm % 128 || r->dm > 64 * LN_MAX_PER_LANE || r->d_ff <= 0 || r->d_ff % 128)
    return set_error(MOQE_E_SHAPE, "%s: d=%d must be a multiple of 64, dm=%d and d_ff=%d multiples of 128, dm <= %d", who, r->d,
                     r->dm, r->d_ff, 64 * LN_MAX_PER_LANE);
  if (r->n_heads <= 0 || r->dm % r->n_heads) return set_error(MOQE_E_SHAPE, "%s: %d heads do not divide dm=%d", who, r->n_heads, r->dm);
  const int dh = r->dm / r->n_heads;
  if (dh != 16 && dh != 32 && dh != 64 && dh != 128)
    return set_error(MOQE_E_SHAPE, "%s: head width %d must be 16, 32, 64 or 128", who, dh);
  if (r->head.d != r->dm) return set_error(MOQE_E_SHAPE, "%s: the MLP head takes %d features, dm is %d", who, r->head.d, r->dm);
  return MOQE_OK;
}

size_t route_nlp_ws_bytes(int S, int T, const moqe_nlp_router& r) { return nlp_layout(S, T, r).total; }

int32_t launch_route_nlp(const void* x, int S, int T, const moqe_nlp_router& r, int32_t* idx, float* logits, void* ws, hipStream_t st) {
  const NlpLayout L = nlp_layout(S, T, r);
  uint8_t* p = static_cast<uint8_t*>(ws);
  auto b16 = [&](size_t off) { return reinterpret_cast<uint16_t*>(p + off); };
  auto f32 = [&](size_t off) { return reinterpret_cast<float*>(p + off); };
  const int M = S * T, dm = r.dm, dff = r.d_ff;
  int32_t rc;
  if (nlp_whole_rows(M, r.d, dm, dff)) {
    const size_t w_at[7] = {L.w_in, L.wqkv1, L.wo1, L.wff1, L.wff2, L.wqkv2, L.wo2};
    if ((rc = launch_route_nlp_rows(x, S, T, r, p, w_at, f32(L.t32a), f32(L.t32b), b16(L.t16b), f32(L.qkv), f32(L.pooled), st))) return rc;
    return launch_route_features(f32(L.pooled), S, r.head, idx, logits, p + L.head, st);
  }
  {
    CvtSegs sg;
    memset(&sg, 0, sizeof(sg));
    const float* src[7] = {r.w_in, r.wqkv1, r.wo1, r.w_ff1, r.w_ff2, r.wqkv2, r.wo2};
    const size_t dst[7] = {L.w_in, L.wqkv1, L.wo1, L.wff1, L.wff2, L.wqkv2, L.wo2};
    const long long cnt[7] = {(long long)dm * r.d, 3ll * dm * dm, (long long)dm * dm, (long long)dff * dm, (long long)dff * dm,
                              3ll * dm * dm, (long long)dm * dm};
    sg.n = 7;
    for (int i = 0; i < 7; ++i) {
      sg.src[i] = src[i];
      sg.dst[i] = b16(dst[i]);
      sg.first[i + 1] = sg.first[i] + cnt[i] / 4;          // every count is a multiple of 64
    }
    ProfileScope ps(MOQE_PK_ROUTE, st);
    const long long blocks = (sg.first[7] + 255) / 256;
    hipLaunchKernelGGL(k_to_bf16, dim3(unsigned(blocks < 2048 ? blocks : 2048)), dim3(256), 0, st, sg);
    rc = check_launch("route_nlp(parameters)");
    if (rc) return rc;
  }
  const uint16_t* xb = static_cast<const uint16_t*>(x);
  // u = x W_in^T + b_in                                             u: t32a / t16a
  if ((rc = lin(xb, b16(L.w_in), r.b_in, nullptr, f32(L.t32a), b16(L.t16a), M, dm, r.d, false, f32(L.part), st))) return rc;
  // encoder layer: v = LN1(u + attention(u))                         v: t32c / t16a
  if ((rc = lin(b16(L.t16a), b16(L.wqkv1), r.bqkv1, nullptr, f32(L.qkv), nullptr, M, 3 * dm, dm, false, f32(L.part), st))) return rc;
  if ((rc = launch_nlp_attention(f32(L.qkv), b16(L.t16b), S, T, dm, r.n_heads, st))) return rc;
  if ((rc = lin(b16(L.t16b), b16(L.wo1), r.bo1, f32(L.t32a), f32(L.t32b), nullptr, M, dm, dm, false, f32(L.part), st))) return rc;
  if ((rc = layer_norm(f32(L.t32b), r.ln1_g, r.ln1_b, M, dm, f32(L.t32c), b16(L.t16a), st))) return rc;
  //                w = LN2(v + W2 relu(W1 v + b1) + b2)              w: t32a / t16a
  if ((rc = lin(b16(L.t16a), b16(L.wff1), r.b_ff1, nullptr, nullptr, b16(L.hid), M, dff, dm, true, f32(L.part), st))) return rc;
  if ((rc = lin(b16(L.hid), b16(L.wff2), r.b_ff2, f32(L.t32c), f32(L.t32b), nullptr, M, dm, dff, false, f32(L.part), st))) return rc;
  if ((rc = layer_norm(f32(L.t32b), r.ln2_g, r.ln2_b, M, dm, f32(L.t32a), b16(L.t16a), st))) return rc;
  // attention module: z = LN3(w + attention2(w)); z itself is never stored: LN3 and the mean over the tokens take t32b to the pooled vector
  if ((rc = lin(b16(L.t16a), b16(L.wqkv2), r.bqkv2, nullptr, f32(L.qkv), nullptr, M, 3 * dm, dm, false, f32(L.part), st))) return rc;
  if ((rc = launch_nlp_attention(f32(L.qkv), b16(L.t16b), S, T, dm, r.n_heads, st))) return rc;
  if ((rc = lin(b16(L.t16b), b16(L.wo2), r.bo2, f32(L.t32a), f32(L.t32b), nullptr, M, dm, dm, false, f32(L.part), st))) return rc;
  {
    // chunks of a sample's tokens: enough work-groups for two to a CU, at least 32 rows each; their sums go to t32c, which has T rows per
    // sample and is no longer needed (with one chunk they go to the pooled vector)
    int chunks = (512 + S - 1) / S;
    if (chunks > T / 32) chunks = T / 32;
    if (chunks < 1) chunks = 1;
    const int rows = (T + chunks - 1) / chunks;
    chunks = (T + rows - 1) / rows;
    float* part = chunks == 1 ? f32(L.pooled) : f32(L.t32c);
    ProfileScope ps(MOQE_PK_ROUTE, st);
    if (dm <= 512) hipLaunchKernelGGL((k_ln_pool<8, 16>), dim3(chunks, S), dim3(1024), 0, st, f32(L.t32b), r.ln3_g, r.ln3_b, T, dm, rows, part);
    else if (dm <= 1024) hipLaunchKernelGGL((k_ln_pool<16, 8>), dim3(chunks, S), dim3(512), 0, st, f32(L.t32b), r.ln3_g, r.ln3_b, T, dm, rows, part);
    else hipLaunchKernelGGL((k_ln_pool<32, 4>), dim3(chunks, S), dim3(256), 0, st, f32(L.t32b), r.ln3_g, r.ln3_b, T, dm, rows, part);
    if (chunks > 1)
      hipLaunchKernelGGL(k_pool_f32, dim3(unsigned((size_t(S) * dm + 255) / 256)), dim3(256), 0, st, part, f32(L.pooled), S, chunks, dm, T);
    if ((rc = check_launch("route_nlp(pool)"))) return rc;
  }
  return launch_route_features(f32(L.pooled), S, r.head, idx, logits, p + L.head, st);
}

}  // namespace moqe
