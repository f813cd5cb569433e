// The NLP router model (MoQE Section 3.2) for widths of up to 384 and more than 512 token rows: everything between its two attentions works
// on whole token rows, so a work-group keeps 16 RB rows and takes them through a chain of products, LayerNorms and residuals
// without leaving the CU:
//   k_rows_in    u = x W_in^T + b, stored;  q, k, v of the encoder's attention = u W_qkv^T + b
//   k_rows_mid   v = LN1(u + att Wo^T + b);  w = LN2(v + W2 relu(W1 v + b1) + b2), stored;  q, k, v of the second attention
//   k_rows_out   z = LN3(w + att2 Wo^T + b), summed over the rows of each sample (k_rows_pool adds the tiles and divides)
//   k_to_operands  the parameter matrices as bf16 in matrix-core operand order
// One launch per product and LayerNorm moved eight intermediates out and in, 25 to 100 MB apiece on 32768 rows of 384, and at a few
// thousand rows cost mostly launches, fills and drains.  Here the rows sit in LDS as bf16 operands (16-byte units XOR-swizzled by the
// row: 16 rows meet all banks).
// Weights never touch LDS: each of the eight waves owns 16 NB of the 128 NB columns of a product, so a weight is needed by one wave only,
// and k_to_operands lays it out so that a 16 x 32 tile is one coalesced 1 KiB load (L2 holds all matrices), four k-tiles ahead and on
// into the next product's.  A product then has no barrier inside.  Sums run over k in order, as in k_lin; everything but the operands is fp32.
// 32768 rows, 3584 -> 384, feed-forward 1536: k_rows_in 148 us for 185 in two launches, k_rows_mid 161 for 300 in six, k_rows_out 30 for 55
// in two; the call 742 -> 540, with 16384 rows 397 -> 238, 4096 rows 179 -> 136.  What is left is memory (q, k, v in fp32: 151 MB out of
// each of the first two) that the products of one work-group per CU do not cover; storing past the caches was slower (mid 160 -> 168).
#include "bf16_pieces.h"
#include "dispatch_rules.h"
#include "qgemm_device.h"

#include <algorithm>

namespace moqe {

constexpr int RW_THREADS = 512;
typedef __attribute__((address_space(3))) void rw_lds;
typedef float f32x4_any __attribute__((ext_vector_type(4), aligned(4)));   // LayerNorm vectors may lie on any float

// ---- parameters ---------------------------------------------------------------------------------------------------
// Operand order: tiles of 16 rows x 32 columns, row-tile major; lane l of a tile holds row l % 16, columns 8 (l / 16) .. + 7.
constexpr int OPS_MATS = 7;
struct OpsArgs {
  const float* src[OPS_MATS];
  uint32_t dst[OPS_MATS];            // byte offset behind w
  uint32_t kt[OPS_MATS];             // k / 32
  uint32_t first[OPS_MATS + 1];      // index (in units of 8 elements) where matrix i starts
  uint8_t* w;
};
__global__ __launch_bounds__(256) void k_to_operands(const OpsArgs oa) {
  const uint32_t total = oa.first[OPS_MATS];
  for (uint32_t i = blockIdx.x * 256u + threadIdx.x; i < total; i += gridDim.x * 256u) {
    int s = 0;
#pragma unroll
    for (int j = 1; j < OPS_MATS; ++j) s += i >= oa.first[j] ? 1 : 0;
    const uint32_t e = i - oa.first[s], tile = e >> 6, l = e & 63u, kt = oa.kt[s];
    const uint32_t nt = tile / kt, col = (tile - nt * kt) * 32u + (l >> 4) * 8u;
    const float* p = oa.src[s] + size_t(nt * 16u + (l & 15u)) * (size_t(kt) * 32u) + col;
    const float4 a = *reinterpret_cast<const float4*>(p), b = *reinterpret_cast<const float4*>(p + 4);
    u32x4 o;
    o.x = pack_bf16x2(a.x, a.y); o.y = pack_bf16x2(a.z, a.w); o.z = pack_bf16x2(b.x, b.y); o.w = pack_bf16x2(b.z, b.w);
    *reinterpret_cast<u32x4*>(oa.w + oa.dst[s] + size_t(e) * 16u) = o;
  }
}

// ---- pieces -------------------------------------------------------------------------------------------------------
struct RowsArgs {
  const uint8_t* w;                  // operands
  uint32_t o_in, o_qkv, o_wo, o_ff1, o_ff2;       // byte offsets of the matrices a kernel uses
  const float *b_in, *b_qkv, *b_o, *b_ff1, *b_ff2;
  const float *ln_a_g, *ln_a_b, *ln_b_g, *ln_b_b;
  const uint16_t* a;                 // bf16 [M, d] (k_rows_in) or [M, dm]: the rows
  const float* res;                  // fp32 [M, dm], residual
  float* rows;                       // fp32 [M, dm], stored for a later residual (k_rows_out: the sums per sample and tile)
  float* qkv;                        // fp32 [M, 3 dm]
  int M, d, d_ff, T;
};

// where a wave's weights of one product lie: first tile of its first block of 16 columns, bytes from a block to the next
struct WAt { uint32_t at, step; };

static __device__ __forceinline__ void rows_barrier() {      // LDS traffic done; loads to registers stay in flight
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_waitcnt(15 | (7 << 4) | (0 << 8) | (3 << 14));
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
}

struct Lane {
  int wave, lane, lr, lq;
  __device__ __forceinline__ Lane() {
    lane = threadIdx.x & 63;
    wave = __builtin_amdgcn_readfirstlane(int(threadIdx.x) >> 6);
    lr = lane & 15;
    lq = lane >> 4;
  }
};

template <int NB, int RB> struct Rows {
  static constexpr int DM = 128 * NB, TM = 16 * RB, PITCH = DM * 2;
  typedef f32x4 Acc[RB][NB];         // lane (lr, lq): row 16 rb + lr, columns 16 (wave NB + nb) + 4 lq .. + 3
  typedef u32x4 Ring[4][NB];

  static __device__ __forceinline__ WAt weights(uint32_t matrix, uint32_t first_block, uint32_t k_tiles, uint32_t first_kt, int wave) {
    return WAt{matrix + ((first_block + uint32_t(wave) * NB) * k_tiles + first_kt) * 1024u, k_tiles * 1024u};
  }
  static __device__ __forceinline__ void clear(Acc& acc) {
#pragma unroll
    for (int rb = 0; rb < RB; ++rb)
#pragma unroll
      for (int nb = 0; nb < NB; ++nb) acc[rb][nb] = f32x4{0.f, 0.f, 0.f, 0.f};
  }
  static __device__ __forceinline__ void fill(Ring& ring, buf_rsrc w, WAt s, const Lane& ln) {
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int nb = 0; nb < NB; ++nb) ring[i][nb] = buf_load128(w, ln.lane * 16, s.at + uint32_t(nb) * s.step + uint32_t(i) * 1024u);
  }
  // acc += rows (LDS) x weights over k = DM; the ring holds the first four k-tiles and leaves with the next product's
  static __device__ __forceinline__ void product(Acc& acc, Ring& ring, const uint8_t* rows, buf_rsrc w, WAt cur, WAt next, const Lane& ln) {
    uint32_t a_off[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) a_off[i] = uint32_t(ln.lr * PITCH + ((i * 4 + ln.lq) ^ ln.lr) * 16);
    auto read = [&](bf16x8 (&af)[RB], int g, int i) {
#pragma unroll
      for (int rb = 0; rb < RB; ++rb)
        af[rb] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const u32x4*>(rows + rb * 16 * PITCH + g * 256 + a_off[i]));
    };
    bf16x8 af[2][RB];                // a k-tile's rows are read while the one before is multiplied
    read(af[0], 0, 0);
#pragma unroll 1
    for (int g = 0; g < NB; ++g) {
      const WAt s = g + 1 < NB ? WAt{cur.at + uint32_t(g + 1) * 4096u, cur.step} : next;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        read(af[(i + 1) & 1], i < 3 ? g : min(g + 1, NB - 1), (i + 1) & 3);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int nb = 0; nb < NB; ++nb)
#pragma unroll
          for (int rb = 0; rb < RB; ++rb) acc[rb][nb] = mfma_bf16(ring[i][nb], af[i & 1][rb], acc[rb][nb]);
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) ring[i][nb] = buf_load128(w, ln.lane * 16, s.at + uint32_t(nb) * s.step + uint32_t(i) * 1024u);
        __builtin_amdgcn_sched_barrier(0);
      }
    }
  }
  static __device__ __forceinline__ int col(int nb, const Lane& ln) { return (ln.wave * NB + nb) * 16 + 4 * ln.lq; }
  static __device__ __forceinline__ void add_bias(Acc& acc, const float* bias, const Lane& ln) {
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) {
      const f32x4 b = *reinterpret_cast<const f32x4*>(bias + col(nb, ln));
#pragma unroll
      for (int rb = 0; rb < RB; ++rb) acc[rb][nb] = acc[rb][nb] + b;
    }
  }
  static __device__ __forceinline__ void load_rows(Acc& v, const float* src, int m0, int M, const Lane& ln) {
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) {
      const float* p = src + size_t(min(m0 + rb * 16 + ln.lr, M - 1)) * DM;
#pragma unroll
      for (int nb = 0; nb < NB; ++nb) v[rb][nb] = *reinterpret_cast<const f32x4*>(p + col(nb, ln));
    }
  }
  static __device__ __forceinline__ void store_rows(const Acc& v, float* dst, int ld, int m0, int M, const Lane& ln) {
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) {
      if (m0 + rb * 16 + ln.lr >= M) continue;
      float* p = dst + size_t(m0 + rb * 16 + ln.lr) * ld;
#pragma unroll
      for (int nb = 0; nb < NB; ++nb) *reinterpret_cast<f32x4*>(p + col(nb, ln)) = v[rb][nb];
    }
  }
  static __device__ __forceinline__ void to_operands(const Acc& v, uint8_t* rows, const Lane& ln) {
#pragma unroll
    for (int rb = 0; rb < RB; ++rb)
#pragma unroll
      for (int nb = 0; nb < NB; ++nb) {
        const int unit = (ln.wave * NB + nb) * 2 + (ln.lq >> 1);
        uint2 o;
        o.x = pack_bf16x2(v[rb][nb].x, v[rb][nb].y);
        o.y = pack_bf16x2(v[rb][nb].z, v[rb][nb].w);
        *reinterpret_cast<uint2*>(rows + (rb * 16 + ln.lr) * PITCH + (unit ^ ln.lr) * 16 + (ln.lq & 1) * 8) = o;
      }
  }
  // bf16 rows m0 .. of [M, DM] into LDS; rows past the end repeat the last one
  static __device__ __forceinline__ void fetch(uint8_t* rows, const uint16_t* src, int m0, int M) {
    constexpr int UNITS = PITCH / 16;
#pragma unroll
    for (int i = 0; i < (TM * UNITS + RW_THREADS - 1) / RW_THREADS; ++i) {
      const int id = int(threadIdx.x) + i * RW_THREADS;
      if (id < TM * UNITS) {
        const int r = id / UNITS, u = id % UNITS;
        const u32x4 v = *reinterpret_cast<const u32x4*>(src + size_t(min(m0 + r, M - 1)) * DM + u * 8);
        *reinterpret_cast<u32x4*>(rows + r * PITCH + (u ^ (r & 15)) * 16) = v;
      }
    }
  }
  // Sums over the columns of each row: a wave's share by lane exchange, the eight shares in wave order.  One barrier.
  static __device__ __forceinline__ void row_sums(const float (&mine)[RB], float (&out)[RB], float* red, const Lane& ln) {
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) {
      float v = mine[rb];
      v += __shfl_xor(v, 16);
      v += __shfl_xor(v, 32);
      if (ln.lq == 0) red[(rb * 16 + ln.lr) * 8 + ln.wave] = v;
    }
    rows_barrier();
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) {
      const f32x4 a = *reinterpret_cast<const f32x4*>(red + (rb * 16 + ln.lr) * 8), b = *reinterpret_cast<const f32x4*>(red + (rb * 16 + ln.lr) * 8 + 4);
      out[rb] = ((((((a.x + a.y) + a.z) + a.w) + b.x) + b.y) + b.z) + b.w;
    }
  }
  // red: [2][TM * 8].  Two barriers: every wave has left the product before, and the second half of red is free for the next call.
  static __device__ __forceinline__ void layer_norm(Acc& v, const float* g, const float* b, float* red, const Lane& ln) {
    float s[RB], mu[RB], sq[RB];
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) {
      s[rb] = 0.f;
#pragma unroll
      for (int nb = 0; nb < NB; ++nb) s[rb] += (v[rb][nb].x + v[rb][nb].y) + (v[rb][nb].z + v[rb][nb].w);
    }
    row_sums(s, mu, red, ln);
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) {
      mu[rb] = mu[rb] / float(DM);
      s[rb] = 0.f;
#pragma unroll
      for (int nb = 0; nb < NB; ++nb)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const float d = v[rb][nb][r] - mu[rb];
          s[rb] += d * d;
        }
    }
    row_sums(s, sq, red + TM * 8, ln);
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) {
      const f32x4 gg = *reinterpret_cast<const f32x4_any*>(g + col(nb, ln)), bb = *reinterpret_cast<const f32x4_any*>(b + col(nb, ln));
#pragma unroll
      for (int rb = 0; rb < RB; ++rb) {
        const float rstd = 1.0f / sqrtf(sq[rb] / float(DM) + 1e-5f);
#pragma unroll
        for (int r = 0; r < 4; ++r) v[rb][nb][r] = (v[rb][nb][r] - mu[rb]) * rstd * gg[r] + bb[r];
      }
    }
  }
  // queries, keys and values of the rows in LDS; the ring holds the first tiles of the queries' weights
  static __device__ __forceinline__ void qkv(Ring& ring, const uint8_t* rows, buf_rsrc w, const RowsArgs& ra, int m0, const Lane& ln) {
#pragma unroll 1
    for (int j = 0; j < 3; ++j) {
      Acc acc;
      clear(acc);
      const WAt cur = weights(ra.o_qkv, uint32_t(j) * 8 * NB, 4 * NB, 0, ln.wave);
      product(acc, ring, rows, w, cur, weights(ra.o_qkv, uint32_t(min(j + 1, 2)) * 8 * NB, 4 * NB, 0, ln.wave), ln);
      add_bias(acc, ra.b_qkv + j * DM, ln);
      store_rows(acc, ra.qkv + j * DM, 3 * DM, m0, ra.M, ln);
    }
  }
};

// ---- x -> u, q k v -------------------------------------------------------------------------------------------------
// The long product (k = d): rows of x stream through four LDS buffers of 128 columns, loaded directly, three ahead, one barrier per buffer;
// the ring of weights is eight k-tiles deep, because loads return in order and a wave that waits for its next weights waits for the
// rows requested before them.
template <int NB, int RB>
__global__ __launch_bounds__(RW_THREADS, 2) void k_rows_in(const RowsArgs ra) {
  typedef Rows<NB, RB> R;
  __shared__ __align__(1024) uint8_t buf0[R::TM * 256], buf1[R::TM * 256], buf2[R::TM * 256], buf3[R::TM * 256];
  __shared__ __align__(1024) uint8_t tile[R::TM * R::PITCH];
  const Lane ln;
  const int m0 = int(blockIdx.x) * R::TM;
  const buf_rsrc w = blob_rsrc(ra.w);
  const int KT = ra.d >> 5, C = (KT + 3) >> 2;
  const uint32_t pitch = uint32_t(ra.d) * 2u;
  const int rows = min(R::TM, ra.M - m0);
  const buf_rsrc x = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t*>(ra.a + size_t(m0) * ra.d), 0, uint32_t(rows) * pitch, 0x00020000);
  // A request fills 1 KiB: four rows of a buffer.  With 16 rows there are four requests, made by two waves each (the same bytes).
  constexpr int REQ = RB >= 2 ? RB / 2 : 1;
  uint32_t x_off[REQ], x_back[REQ];
  int x_dst[REQ];
#pragma unroll
  for (int i = 0; i < REQ; ++i) {
    const int q = (i * 8 + ln.wave) % (4 * RB), row = q * 4 + (ln.lane >> 4);
    const uint32_t unit = uint32_t((ln.lane & 15) ^ (row & 15));
    x_off[i] = uint32_t(min(row, rows - 1)) * pitch + unit * 16u;
    x_back[i] = (ra.d & 64) && unit >= 8u ? 128u : 0u;     // d = 64 (mod 128): the second half of the last buffer, which is not multiplied, repeats the first
    x_dst[i] = q * 1024;
  }
  auto request = [&](uint8_t* buf, int c) {
#pragma unroll
    for (int i = 0; i < REQ; ++i)
      __builtin_amdgcn_raw_ptr_buffer_load_lds(x, (rw_lds*)(buf + x_dst[i]), 16, int(c >= C - 1 ? x_off[i] - x_back[i] : x_off[i]),
                                               min(c, C - 1) * 256, 0, 0);
  };
  const WAt win = R::weights(ra.o_in, 0, uint32_t(KT), 0, ln.wave);
  u32x4 ring[8][NB];
  auto weights = [&](int slot, int kt) {
#pragma unroll
    for (int nb = 0; nb < NB; ++nb)
      ring[slot][nb] = buf_load128(w, ln.lane * 16, win.at + uint32_t(nb) * win.step + uint32_t(min(kt, KT - 1)) * 1024u);
  };
  uint32_t a_off[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) a_off[i] = uint32_t(ln.lr * 256 + ((i * 4 + ln.lq) ^ ln.lr) * 16);
  typename R::Acc acc;
  R::clear(acc);
  auto chunk = [&](int c, int half, const uint8_t* cur, uint8_t* next, bool full) {
    // At most the requests of the two chunks after this one and the weights asked for since are still in flight.
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_waitcnt(((2 * REQ + 8 * NB) & 15) | (7 << 4) | (0 << 8) | (((2 * REQ + 8 * NB) >> 4) << 14));
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
    request(next, c + 3);                                  // last read a chunk ago, before the barrier
    __builtin_amdgcn_sched_barrier(0);
    bf16x8 af[2][RB];
    auto read = [&](int i) {
#pragma unroll
      for (int rb = 0; rb < RB; ++rb) af[i & 1][rb] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const u32x4*>(cur + rb * 16 * 256 + a_off[i]));
    };
    read(0);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int slot = half * 4 + i;
      if (i < 3) read(i + 1);
      __builtin_amdgcn_sched_barrier(0);
      if (full || i < 2 || c * 4 + i < KT) {               // d is a multiple of 64
#pragma unroll
        for (int nb = 0; nb < NB; ++nb)
#pragma unroll
          for (int rb = 0; rb < RB; ++rb) acc[rb][nb] = mfma_bf16(ring[slot][nb], af[i & 1][rb], acc[rb][nb]);
      }
      weights(slot, c * 4 + i + 8);
      __builtin_amdgcn_sched_barrier(0);
    }
  };
  request(buf0, 0);
  request(buf1, 1);
  request(buf2, 2);
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int i = 0; i < 8; ++i) weights(i, i);
  __builtin_amdgcn_sched_barrier(0);
  int c = 0;
#pragma unroll 1
  for (; c + 4 <= (KT >> 2); c += 4) {
    chunk(c, 0, buf0, buf3, true);
    chunk(c + 1, 1, buf1, buf0, true);
    chunk(c + 2, 0, buf2, buf1, true);
    chunk(c + 3, 1, buf3, buf2, true);
  }
  if (c < C) chunk(c, 0, buf0, buf3, false);               // uniform over the grid
  if (c + 1 < C) chunk(c + 1, 1, buf1, buf0, false);
  if (c + 2 < C) chunk(c + 2, 0, buf2, buf1, false);
  if (c + 3 < C) chunk(c + 3, 1, buf3, buf2, false);
  typename R::Ring wring;
  R::fill(wring, w, R::weights(ra.o_qkv, 0, 4 * NB, 0, ln.wave), ln);
  R::add_bias(acc, ra.b_in, ln);
  R::to_operands(acc, tile, ln);
  R::store_rows(acc, ra.rows, R::DM, m0, ra.M, ln);
  rows_barrier();
  R::qkv(wring, tile, w, ra, m0, ln);
  __builtin_amdgcn_s_waitcnt(0);                           // requests into LDS past the last chunk: none outlives the work-group
}

// The same with 128 rows a work-group (rows_in_128() says when): they meet a weight of the long product in two halves, where 64 bring in as many bytes per matrix
// operation as a CU's vector memory path carries (24 KiB of weights per k-tile of 384 clocks).  Three buffers, two chunks ahead, which last as
// long as four of the others; the ring is four k-tiles deep.  q, k and v are made of 64 rows at a time.  Eleven registers are spilled (44 bytes of scratch): stored ahead of
// the long product and read behind it, but for 16 bytes in a loop of the q, k, v part.  Were one read inside the product, its counted waits would only wait for more.
template <int NB>
__global__ __launch_bounds__(RW_THREADS, 2) void k_rows_in_128(const RowsArgs ra) {
  constexpr int RB = 8, REQ = 4;
  typedef Rows<NB, 4> R;
  __shared__ __align__(1024) uint8_t buf0[16 * RB * 256], buf1[16 * RB * 256], buf2[16 * RB * 256];
  __shared__ __align__(1024) uint8_t tile[R::TM * R::PITCH];
  const Lane ln;
  const int m0 = int(blockIdx.x) * (16 * RB);
  const buf_rsrc w = blob_rsrc(ra.w);
  const int KT = ra.d >> 5, C = (KT + 3) >> 2;
  const uint32_t pitch = uint32_t(ra.d) * 2u;
  const int rows = min(16 * RB, ra.M - m0);
  const buf_rsrc x = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t*>(ra.a + size_t(m0) * ra.d), 0, uint32_t(rows) * pitch, 0x00020000);
  uint32_t x_off[REQ], x_back;
  const int row0 = ln.wave * 4 + (ln.lane >> 4);              // of request 0; 32 rows from one to the next
  const uint32_t unit = uint32_t((ln.lane & 15) ^ (row0 & 15));
  x_back = (ra.d & 64) && unit >= 8u ? 128u : 0u;             // as above
#pragma unroll
  for (int i = 0; i < REQ; ++i) x_off[i] = uint32_t(min(row0 + 32 * i, rows - 1)) * pitch + unit * 16u;
  auto request = [&](uint8_t* buf, int c) {
#pragma unroll
    for (int i = 0; i < REQ; ++i)
      __builtin_amdgcn_raw_ptr_buffer_load_lds(x, (rw_lds*)(buf + (i * 8 + ln.wave) * 1024), 16, int(c >= C - 1 ? x_off[i] - x_back : x_off[i]), min(c, C - 1) * 256, 0, 0);
  };
  const WAt win = R::weights(ra.o_in, 0, uint32_t(KT), 0, ln.wave);
  u32x4 ring[4][NB];
  auto weights = [&](int slot, int kt) {
#pragma unroll
    for (int nb = 0; nb < NB; ++nb)
      ring[slot][nb] = buf_load128(w, ln.lane * 16, win.at + uint32_t(nb) * win.step + uint32_t(min(kt, KT - 1)) * 1024u);
  };
  uint32_t a_off[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) a_off[i] = uint32_t(ln.lr * 256 + ((i * 4 + ln.lq) ^ ln.lr) * 16);
  f32x4 acc[RB][NB];
#pragma unroll
  for (int rb = 0; rb < RB; ++rb)
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) acc[rb][nb] = f32x4{0.f, 0.f, 0.f, 0.f};
  auto chunk = [&](int c, const uint8_t* cur, uint8_t* next, bool full) {
    // At most the requests of the chunk after this one and the weights asked for since are still in flight.
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_waitcnt(((REQ + 4 * NB) & 15) | (7 << 4) | (0 << 8) | (((REQ + 4 * NB) >> 4) << 14));
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
    request(next, c + 2);                                     // last read a chunk ago, before the barrier
    __builtin_amdgcn_sched_barrier(0);
    bf16x8 af[2][4];                                          // half a k-tile's rows are read while the half before is multiplied
    auto read = [&](int q) {
#pragma unroll
      for (int rb = 0; rb < 4; ++rb)
        af[q & 1][rb] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const u32x4*>(cur + ((q & 1) * 4 + rb) * 16 * 256 + a_off[q >> 1]));
    };
    read(0);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        if (i * 2 + h < 7) read(i * 2 + h + 1);
        __builtin_amdgcn_sched_barrier(0);
        if (full || i < 2 || c * 4 + i < KT) {                // d is a multiple of 64
#pragma unroll
          for (int nb = 0; nb < NB; ++nb)
#pragma unroll
            for (int rb = 0; rb < 4; ++rb) acc[h * 4 + rb][nb] = mfma_bf16(ring[i][nb], af[h][rb], acc[h * 4 + rb][nb]);
        }
        if (h == 1) weights(i, c * 4 + i + 4);
        __builtin_amdgcn_sched_barrier(0);
      }
    }
  };
  request(buf0, 0);
  request(buf1, 1);
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int i = 0; i < 4; ++i) weights(i, i);
  __builtin_amdgcn_sched_barrier(0);
  int c = 0;
#pragma unroll 1
  for (; c + 3 <= (KT >> 2); c += 3) {
    chunk(c, buf0, buf2, true);
    chunk(c + 1, buf1, buf0, true);
    chunk(c + 2, buf2, buf1, true);
  }
  if (c < C) chunk(c, buf0, buf2, false);                     // uniform over the grid
  if (c + 1 < C) chunk(c + 1, buf1, buf0, false);
  if (c + 2 < C) chunk(c + 2, buf2, buf1, false);
  __builtin_amdgcn_s_waitcnt(0);                              // requests into LDS past the last chunk: none outlives the work-group
#pragma unroll 1
  for (int half = 0; half < 2; ++half) {
    if (half * 64 >= rows) break;                             // uniform
    typename R::Acc v;
    if (half == 0) {
#pragma unroll
      for (int rb = 0; rb < 4; ++rb)
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) v[rb][nb] = acc[rb][nb];
    } else {
#pragma unroll
      for (int rb = 0; rb < 4; ++rb)
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) v[rb][nb] = acc[4 + rb][nb];
    }
    typename R::Ring wring;
    R::fill(wring, w, R::weights(ra.o_qkv, 0, 4 * NB, 0, ln.wave), ln);
    R::add_bias(v, ra.b_in, ln);
    rows_barrier();                                           // the first half's rows have been read
    R::to_operands(v, tile, ln);
    R::store_rows(v, ra.rows, R::DM, m0 + half * 64, ra.M, ln);
    rows_barrier();
    R::qkv(wring, tile, w, ra, m0 + half * 64, ln);
  }
}

// ---- attention, u -> w, q k v ----------------------------------------------------------------------------------------
template <int NB, int RB>
__global__ __launch_bounds__(RW_THREADS, 2) void k_rows_mid(const RowsArgs ra) {
  typedef Rows<NB, RB> R;
  __shared__ __align__(1024) uint8_t tile[R::TM * R::PITCH], hid[R::TM * R::PITCH];
  __shared__ __align__(16) float red[2 * R::TM * 8];
  const Lane ln;
  const int m0 = int(blockIdx.x) * R::TM;
  const buf_rsrc w = blob_rsrc(ra.w);
  typename R::Ring ring;
  typename R::Acc v, acc;
  R::fetch(tile, ra.a, m0, ra.M);
  const WAt wo = R::weights(ra.o_wo, 0, 4 * NB, 0, ln.wave);
  R::fill(ring, w, wo, ln);
  R::load_rows(v, ra.res, m0, ra.M, ln);
  rows_barrier();
  const int chunks = ra.d_ff / R::DM;
  const uint32_t kt_ff = uint32_t(ra.d_ff) / 32u;
  auto ff1 = [&](int c) { return R::weights(ra.o_ff1, uint32_t(c) * 8 * NB, 4 * NB, 0, ln.wave); };
  auto ff2 = [&](int c) { return R::weights(ra.o_ff2, 0, kt_ff, uint32_t(c) * 4 * NB, ln.wave); };
  R::clear(acc);
  R::product(acc, ring, tile, w, wo, ff1(0), ln);
  R::add_bias(acc, ra.b_o, ln);
#pragma unroll
  for (int rb = 0; rb < RB; ++rb)
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) v[rb][nb] = acc[rb][nb] + v[rb][nb];
  R::layer_norm(v, ra.ln_a_g, ra.ln_a_b, red, ln);
  R::to_operands(v, tile, ln);
  R::clear(acc);
#pragma unroll 1
  for (int c = 0; c < chunks; ++c) {
    typename R::Acc h;
    R::clear(h);
    rows_barrier();                                        // the rows are there, and hid has been read
    R::product(h, ring, tile, w, ff1(c), ff2(c), ln);
    R::add_bias(h, ra.b_ff1 + c * R::DM, ln);
#pragma unroll
    for (int rb = 0; rb < RB; ++rb)
#pragma unroll
      for (int nb = 0; nb < NB; ++nb)
#pragma unroll
        for (int r = 0; r < 4; ++r) h[rb][nb][r] = fmaxf(h[rb][nb][r], 0.f);
    R::to_operands(h, hid, ln);
    rows_barrier();
    R::product(acc, ring, hid, w, ff2(c), c + 1 < chunks ? ff1(c + 1) : R::weights(ra.o_qkv, 0, 4 * NB, 0, ln.wave), ln);
  }
  R::add_bias(acc, ra.b_ff2, ln);
#pragma unroll
  for (int rb = 0; rb < RB; ++rb)
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) v[rb][nb] = acc[rb][nb] + v[rb][nb];
  R::layer_norm(v, ra.ln_b_g, ra.ln_b_b, red, ln);
  R::to_operands(v, tile, ln);
  R::store_rows(v, ra.rows, R::DM, m0, ra.M, ln);
  rows_barrier();
  R::qkv(ring, tile, w, ra, m0, ln);
}

// ---- second attention, w -> sums of LN3 rows per sample ------------------------------------------------------------
// Tile t's share of sample s goes to row s + t of `rows`: along the rows of the batch s, t or both go up, so no two shares meet.
template <int NB, int RB>
__global__ __launch_bounds__(RW_THREADS, 2) void k_rows_out(const RowsArgs ra) {
  typedef Rows<NB, RB> R;
  constexpr int LD = R::DM + 4;
  __shared__ __align__(1024) uint8_t tile[R::TM * LD * 4];  // bf16 rows, then the normalized fp32 rows
  __shared__ __align__(16) float red[2 * R::TM * 8];
  const Lane ln;
  const int m0 = int(blockIdx.x) * R::TM;
  const buf_rsrc w = blob_rsrc(ra.w);
  typename R::Ring ring;
  typename R::Acc v, acc;
  R::fetch(tile, ra.a, m0, ra.M);
  const WAt wo = R::weights(ra.o_wo, 0, 4 * NB, 0, ln.wave);
  R::fill(ring, w, wo, ln);
  R::load_rows(v, ra.res, m0, ra.M, ln);
  rows_barrier();
  R::clear(acc);
  R::product(acc, ring, tile, w, wo, wo, ln);
  R::add_bias(acc, ra.b_o, ln);
#pragma unroll
  for (int rb = 0; rb < RB; ++rb)
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) v[rb][nb] = acc[rb][nb] + v[rb][nb];
  R::layer_norm(v, ra.ln_a_g, ra.ln_a_b, red, ln);
  float* z = reinterpret_cast<float*>(tile);
#pragma unroll
  for (int rb = 0; rb < RB; ++rb)
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) *reinterpret_cast<f32x4*>(z + (rb * 16 + ln.lr) * LD + R::col(nb, ln)) = v[rb][nb];
  rows_barrier();
  const int c = threadIdx.x;
  if (c >= R::DM) return;
  const int end = min(m0 + R::TM, ra.M);
  int s = m0 / ra.T;
  for (int m = m0; m < end; ++s) {
    const int stop = int(min((long long)(s + 1) * ra.T, (long long)end));
    float sum = 0.f;
#pragma unroll 8
    for (; m < stop; ++m) sum += z[(m - m0) * LD + c];
    ra.rows[(size_t(s) + blockIdx.x) * R::DM + c] = sum;
  }
}

// pooled[s][c] = (the tiles' shares of sample s, in order) / T
__global__ __launch_bounds__(256) void k_rows_pool(const float* __restrict__ part, float* __restrict__ pooled, int S, int T, int tm, int dm) {
  const long long i = (long long)blockIdx.x * 256 + threadIdx.x;
  if (i >= (long long)S * dm) return;
  const int s = int(i / dm), c = int(i % dm);
  const int t0 = int((long long)s * T / tm), t1 = int(((long long)(s + 1) * T - 1) / tm);
  const float* p = part + (size_t(s) + t0) * dm + c;
  float v = p[0];
#pragma unroll 4
  for (int t = t0 + 1; t <= t1; ++t) v += p[size_t(t - t0) * dm];
  pooled[i] = __fdiv_rn(v, float(T));
}

// ---- host side -------------------------------------------------------------------------------------------------------
namespace {
// A round of 128-row work-groups of k_rows_in takes 1.83 times as long as one of 64 (32768 rows of 3584 at width 384: 132 us for 2 x 72), so it pays where it saves
// every second round: 17000 rows of 2048 303 -> 291 us for the call, 20000 of 4096 391 -> 359, 61440 of 1024 772 -> 758; not 41088 of 3584 588 -> 609.  Width 384:
// at width 128 a CU holds two work-groups of 64 (80 KiB of LDS each); at 256 one, as at 384, but 128 rows were not
// measured there.
bool rows_in_128(int M, int dm) { return dm == 384 && (M + 64 * 256 - 1) / (64 * 256) % 2 == 0; }

template <int NB, int RB>
void launch_stage(int stage, const RowsArgs& ra, hipStream_t st) {
  const dim3 g(unsigned((ra.M + 16 * RB - 1) / (16 * RB))), t(RW_THREADS);
  if constexpr (NB == 3 && RB == 4) {
    if (stage == 0 && rows_in_128(ra.M, 128 * NB)) {
      hipLaunchKernelGGL(k_rows_in_128<NB>, dim3(unsigned((ra.M + 127) / 128)), t, 0, st, ra);
      return;
    }
  }
  if (stage == 0) hipLaunchKernelGGL((k_rows_in<NB, RB>), g, t, 0, st, ra);
  else if (stage == 1) hipLaunchKernelGGL((k_rows_mid<NB, RB>), g, t, 0, st, ra);
  else hipLaunchKernelGGL((k_rows_out<NB, RB>), g, t, 0, st, ra);
}
template <int NB>
void launch_stage(int stage, int rb, const RowsArgs& ra, hipStream_t st) {
  if (rb == 1) launch_stage<NB, 1>(stage, ra, st);
  else if (rb == 2) launch_stage<NB, 2>(stage, ra, st);
  else launch_stage<NB, 4>(stage, ra, st);
}

// Rows per work-group, in blocks of 16: the fewest that the chip takes in one round of a work-group per CU.  More rows share a weight among
// more products, but a work-group's time hardly falls with fewer, so a second round costs more (width 384, the call with 1 / 2 / 4 blocks:
// 2048 rows 101 / 110 / 133 us, 4096 136 / 139 / 162, 6000 191 / 137 / 158, 8192 227 / 158 / 171, 12288 255 / 211 / 164, 32768 957 / 666 / 541).
int row_blocks(int M) { return M <= 16 * 256 ? 1 : (M <= 32 * 256 ? 2 : 4); }
}  // namespace

int32_t launch_route_nlp_rows(const void* x, int S, int T, const moqe_nlp_router& r, uint8_t* w, const size_t (&w_at)[7], float* u, float* wres,
                              uint16_t* att, float* qkv, float* pooled, hipStream_t st) {
  const int M = S * T, dm = r.dm, rb = row_blocks(M);
  int32_t rc;
  {
    OpsArgs oa;
    const float* src[OPS_MATS] = {r.w_in, r.wqkv1, r.wo1, r.w_ff1, r.w_ff2, r.wqkv2, r.wo2};
    const int n[OPS_MATS] = {dm, 3 * dm, dm, r.d_ff, dm, 3 * dm, dm}, k[OPS_MATS] = {r.d, dm, dm, dm, r.d_ff, dm, dm};
    oa.w = w;
    oa.first[0] = 0;
    for (int i = 0; i < OPS_MATS; ++i) {
      oa.src[i] = src[i];
      oa.dst[i] = uint32_t(w_at[i]);
      oa.kt[i] = uint32_t(k[i]) / 32u;
      oa.first[i + 1] = oa.first[i] + uint32_t(size_t(n[i]) * size_t(k[i]) / 8);
    }
    ProfileScope ps(MOQE_PK_ROUTE, st);
    const unsigned blocks = (oa.first[OPS_MATS] + 255u) / 256u;
    hipLaunchKernelGGL(k_to_operands, dim3(std::min(blocks, 2048u)), dim3(256), 0, st, oa);
    if ((rc = check_launch("route_nlp(parameters)"))) return rc;
  }
  auto stage = [&](int which, const RowsArgs& ra) {
    ProfileScope ps(MOQE_PK_ROUTE, st);
    if (dm == 128) launch_stage<1>(which, rb, ra, st);
    else if (dm == 256) launch_stage<2>(which, rb, ra, st);
    else launch_stage<3>(which, rb, ra, st);
    return check_launch("route_nlp(rows)");
  };
  RowsArgs ra = {};
  ra.w = w;
  ra.M = M; ra.d = r.d; ra.d_ff = r.d_ff; ra.T = T;
  ra.o_in = uint32_t(w_at[0]); ra.o_qkv = uint32_t(w_at[1]);
  ra.b_in = r.b_in; ra.b_qkv = r.bqkv1;
  ra.a = static_cast<const uint16_t*>(x);
  ra.rows = u; ra.qkv = qkv;
  if ((rc = stage(0, ra))) return rc;
  if ((rc = launch_nlp_attention(qkv, att, S, T, dm, r.n_heads, st))) return rc;
  ra.o_wo = uint32_t(w_at[2]); ra.o_ff1 = uint32_t(w_at[3]); ra.o_ff2 = uint32_t(w_at[4]); ra.o_qkv = uint32_t(w_at[5]);
  ra.b_o = r.bo1; ra.b_ff1 = r.b_ff1; ra.b_ff2 = r.b_ff2; ra.b_qkv = r.bqkv2;
  ra.ln_a_g = r.ln1_g; ra.ln_a_b = r.ln1_b; ra.ln_b_g = r.ln2_g; ra.ln_b_b = r.ln2_b;
  ra.a = att; ra.res = u; ra.rows = wres;
  if ((rc = stage(1, ra))) return rc;
  if ((rc = launch_nlp_attention(qkv, att, S, T, dm, r.n_heads, st))) return rc;
  ra.o_wo = uint32_t(w_at[6]);
  ra.b_o = r.bo2; ra.ln_a_g = r.ln3_g; ra.ln_a_b = r.ln3_b;
  ra.res = wres; ra.rows = qkv;          // S + tiles rows of dm; the projections have been read
  if ((rc = stage(2, ra))) return rc;
  ProfileScope ps(MOQE_PK_ROUTE, st);
  hipLaunchKernelGGL(k_rows_pool, dim3(unsigned((size_t(S) * dm + 255) / 256)), dim3(256), 0, st, qkv, pooled, S, T, 16 * rb, dm);
  return check_launch("route_nlp(pool)");
}

}  // namespace moqe
