// The CV router model (MoQE Section 3.2): per-pixel three-layer MLP with batch normalisation and ReLU -> three
// squeeze-and-excitation basic blocks (16 / 32 / 64 channels, strides 1 / 2 / 2 in the paper) -> multi-head
// self-attention over the positions of the last feature map -> mean -> linear logits -> top-1.
// The whole model has about 0.1 M parameters and a few hundred MFLOP per batch: fp32 arithmetic in LDS, every sum
// in a fixed order.
//
//   k_cv_mlp        the three per-pixel layers (fused path)
//   k_cv_image      everything after them, one work-group per image (fused path)
// Where an image's maps do not fit the LDS, one launch per stage:
//   k_cv_conv       out = [relu] [bn] (conv(in) + bias): 1x1 or 3x3 (padding 1), stride 1 or 2, NHWC, as an
//                   implicit GEMM: 4096 / CT output pixels x CT output channels per work-group (CT = 16, 32, 64),
//                   k in chunks of 32 through LDS, a thread owns 4 pixels x 4 channels
//   k_cv_se_gate    per image: channel means of u, two small linear layers, sigmoid
//   k_cv_se_apply   relu(u * gate + shortcut)
//   k_cv_attn_pool  per image: queries/keys/values, softmax attention per head, mean over positions, output projection
// The logits and the arg-max are the small router's last-layer kernel (route.hip).
#include "bf16_pieces.h"
#include "moqe_internal.h"

#include <algorithm>
#include <cstring>

namespace moqe {

constexpr float CV_BN_EPS = 1e-5f;
constexpr int CV_MAX_C = 64;             // widest layer
constexpr int CV_MAX_POS = 36;           // positions of the last feature map
constexpr int CV_MAX_DH = 16;            // head width
constexpr int CV_LDS_MAX = 160 * 1024;

struct CvConvArgs {
  const void* in;          // [S, hi, wi, cin], bf16 or fp32
  const float* w;          // [cout, taps, cin]
  const float* bias;       // [cout] or NULL
  const float *bn_g, *bn_o, *bn_m, *bn_v;   // all NULL: no normalisation
  float* out;              // [S, ho, wo, cout]
  int in_bf16, S, hi, wi, cin, ho, wo, cout, taps, stride, relu;
};

// CT = output channels per work-group (16, 32 or 64); the work-group takes 4096 / CT output pixels, a thread 4 x 4.
// Both operands are staged four channels at a time (cin is a multiple of 4, so a group of four never straddles a tap).
template <int CT>
__global__ __launch_bounds__(256) void k_cv_conv(const CvConvArgs a) {
  constexpr int PT = 4096 / CT;                    // pixels per work-group
  constexpr int CG = CT / 4;                       // thread groups along the output channels
  constexpr int PI = PT / 32;                      // pixels a thread stages per chunk
  __shared__ __align__(16) float As[32][PT];       // [k][pixel]
  __shared__ __align__(16) float Ws[32][CT];       // [k][output channel]
  const int tid = threadIdx.x;
  const int pg = tid / CG, cg = tid % CG;
  const int M = a.S * a.ho * a.wo, K = a.taps * a.cin;
  const int p0 = blockIdx.x * PT, c0 = blockIdx.y * CT;
  const int pad = a.taps == 9 ? 1 : 0;
  const int kq = tid & 7, r_l = tid >> 3;          // staging: channels 4 kq .. 4 kq + 3 of the chunk, rows r_l + 32 i
  int s_img[PI], s_iy[PI], s_ix[PI];
#pragma unroll
  for (int i = 0; i < PI; ++i) {
    const int px = p0 + r_l + 32 * i;
    if (px < M) {
      const int s = px / (a.ho * a.wo), rem = px - s * (a.ho * a.wo), oy = rem / a.wo, ox = rem - oy * a.wo;
      s_img[i] = s; s_iy[i] = oy * a.stride - pad; s_ix[i] = ox * a.stride - pad;
    } else {
      s_img[i] = -1; s_iy[i] = 0; s_ix[i] = 0;
    }
  }
  float acc[4][4];
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j) acc[i][j] = 0.f;

  for (int kc = 0; kc < K; kc += 32) {
    const int k = kc + 4 * kq;
    const bool kin = k < K;                         // K is a multiple of 4: the four channels are in or out together
    const int tap = kin ? k / a.cin : 0, c = kin ? k - tap * a.cin : 0;
    const int kh = a.taps == 9 ? tap / 3 : 0, kw = a.taps == 9 ? tap - kh * 3 : 0;
#pragma unroll
    for (int i = 0; i < PI; ++i) {
      const int iy = s_iy[i] + kh, ix = s_ix[i] + kw;
      float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
      if (kin && s_img[i] >= 0 && iy >= 0 && iy < a.hi && ix >= 0 && ix < a.wi) {
        const size_t at = ((size_t(s_img[i]) * a.hi + iy) * a.wi + ix) * a.cin + c;
        if (a.in_bf16) {
          const uint2 b = *reinterpret_cast<const uint2*>(static_cast<const uint16_t*>(a.in) + at);
          v = make_float4(__uint_as_float(b.x << 16), __uint_as_float(b.x & 0xffff0000u), __uint_as_float(b.y << 16),
                          __uint_as_float(b.y & 0xffff0000u));
        } else {
          v = *reinterpret_cast<const float4*>(static_cast<const float*>(a.in) + at);
        }
      }
      const int px_l = r_l + 32 * i;
      As[4 * kq + 0][px_l] = v.x; As[4 * kq + 1][px_l] = v.y; As[4 * kq + 2][px_l] = v.z; As[4 * kq + 3][px_l] = v.w;
    }
#pragma unroll
    for (int i = 0; i < (CT + 31) / 32; ++i) {
      const int co_l = r_l + 32 * i;
      if (co_l < CT) {
        float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
        if (kin && c0 + co_l < a.cout) v = *reinterpret_cast<const float4*>(a.w + size_t(c0 + co_l) * K + k);
        Ws[4 * kq + 0][co_l] = v.x; Ws[4 * kq + 1][co_l] = v.y; Ws[4 * kq + 2][co_l] = v.z; Ws[4 * kq + 3][co_l] = v.w;
      }
    }
    __syncthreads();
#pragma unroll 8
    for (int kk = 0; kk < 32; ++kk) {
      const float4 av = *reinterpret_cast<const float4*>(&As[kk][pg * 4]);
      const float4 wv = *reinterpret_cast<const float4*>(&Ws[kk][cg * 4]);
      const float ar[4] = {av.x, av.y, av.z, av.w}, wr[4] = {wv.x, wv.y, wv.z, wv.w};
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) acc[i][j] = fmaf(ar[i], wr[j], acc[i][j]);
    }
    __syncthreads();
  }
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const int co = c0 + cg * 4 + j;
    if (co >= a.cout) continue;
    const float bv = a.bias ? a.bias[co] : 0.f;
    float mean = 0.f, inv = 1.f, gain = 1.f, off = 0.f;
    if (a.bn_g) {
      mean = a.bn_m[co];
      inv = 1.0f / sqrtf(a.bn_v[co] + CV_BN_EPS);
      gain = a.bn_g[co];
      off = a.bn_o[co];
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int px = p0 + pg * 4 + i;
      if (px >= M) continue;
      float v = acc[i][j] + bv;
      if (a.bn_g) v = (v - mean) * inv * gain + off;
      if (a.relu) v = fmaxf(v, 0.f);
      a.out[size_t(px) * a.cout + co] = v;
    }
  }
}

// gate[s][c] = sigmoid(W2 relu(W1 mean_p u[s][p][:] + b1) + b2)[c]; one work-group per image, C <= 64.
__global__ __launch_bounds__(256) void k_cv_se_gate(const float* __restrict__ u, int P, int C, const float* __restrict__ w1,
                                                     const float* __restrict__ b1, const float* __restrict__ w2,
                                                     const float* __restrict__ b2, float* __restrict__ gate) {
  __shared__ float part[4][CV_MAX_C];
  __shared__ float z[CV_MAX_C];
  __shared__ float hid[CV_MAX_C / 4];
  const int s = blockIdx.x, c = threadIdx.x & 63, q = threadIdx.x >> 6, Cr = C / 4;
  float acc = 0.f;
  if (c < C)
    for (int p = q; p < P; p += 4) acc += u[(size_t(s) * P + p) * C + c];
  part[q][c] = acc;
  __syncthreads();
  if (threadIdx.x < C) z[threadIdx.x] = (((part[0][threadIdx.x] + part[1][threadIdx.x]) + part[2][threadIdx.x]) + part[3][threadIdx.x]) / float(P);
  __syncthreads();
  if (threadIdx.x < Cr) {
    float h = b1[threadIdx.x];
    for (int i = 0; i < C; ++i) h = fmaf(w1[threadIdx.x * C + i], z[i], h);
    hid[threadIdx.x] = fmaxf(h, 0.f);
  }
  __syncthreads();
  if (threadIdx.x < C) {
    float g = b2[threadIdx.x];
    for (int i = 0; i < Cr; ++i) g = fmaf(w2[threadIdx.x * Cr + i], hid[i], g);
    gate[size_t(s) * C + threadIdx.x] = 1.0f / (1.0f + expf(-g));
  }
}

__global__ __launch_bounds__(256) void k_cv_se_apply(const float* __restrict__ u, const float* __restrict__ gate,
                                                      const float* __restrict__ shortcut, float* __restrict__ out, int S, int P, int C) {
  const size_t i = size_t(blockIdx.x) * 256 + threadIdx.x, total = size_t(S) * P * C;
  if (i >= total) return;
  const int c = int(i % size_t(C)), s = int(i / (size_t(P) * C));
  out[i] = fmaxf(fmaf(u[i], gate[size_t(s) * C + c], shortcut[i]), 0.f);
}

// One work-group per image: tokens [P, dm] -> queries, keys, values -> per head softmax(q k^T / sqrt(dh)) v -> mean over
// the positions -> output projection -> pooled[s][dm].  (The mean of projected rows is the projection of the mean row.)
__global__ __launch_bounds__(256) void k_cv_attn_pool(const float* __restrict__ x, int P, int dm, int heads, const float* __restrict__ wqkv,
                                                       const float* __restrict__ bqkv, const float* __restrict__ wo,
                                                       const float* __restrict__ bo, float* __restrict__ pooled) {
  extern __shared__ __align__(16) float cv_lds[];
  float* tok = cv_lds;                       // [P][dm]
  float* qkv = tok + P * dm;                 // [P][3 dm]
  float* att = qkv + P * 3 * dm;             // [P][dm]
  float* mean_att = att + P * dm;            // [dm]
  const int s = blockIdx.x, tid = threadIdx.x, dh = dm / heads;
  const float scale = 1.0f / sqrtf(float(dh));
  for (int i = tid; i < P * dm; i += 256) tok[i] = x[size_t(s) * P * dm + i];
  __syncthreads();
  for (int o = tid; o < P * 3 * dm; o += 256) {
    const int p = o / (3 * dm), j = o - p * 3 * dm;
    float v = bqkv[j];
    for (int c = 0; c < dm; ++c) v = fmaf(tok[p * dm + c], wqkv[j * dm + c], v);
    qkv[o] = v;
  }
  __syncthreads();
  for (int item = tid; item < heads * P; item += 256) {
    const int h = item / P, q = item - h * P;
    const float* qv = qkv + q * 3 * dm + h * dh;
    float mx = -INFINITY;
    for (int k = 0; k < P; ++k) {
      const float* kv = qkv + k * 3 * dm + dm + h * dh;
      float d = 0.f;
      for (int c = 0; c < dh; ++c) d = fmaf(qv[c], kv[c], d);
      mx = fmaxf(mx, d * scale);
    }
    float sum = 0.f, acc[CV_MAX_DH];
#pragma unroll
    for (int c = 0; c < CV_MAX_DH; ++c) acc[c] = 0.f;
    for (int k = 0; k < P; ++k) {
      const float* kv = qkv + k * 3 * dm + dm + h * dh;
      const float* vv = qkv + k * 3 * dm + 2 * dm + h * dh;
      float d = 0.f;
      for (int c = 0; c < dh; ++c) d = fmaf(qv[c], kv[c], d);
      const float e = expf(d * scale - mx);
      sum += e;
#pragma unroll
      for (int c = 0; c < CV_MAX_DH; ++c)
        if (c < dh) acc[c] = fmaf(e, vv[c], acc[c]);
    }
    const float inv = 1.0f / sum;
#pragma unroll
    for (int c = 0; c < CV_MAX_DH; ++c)
      if (c < dh) att[q * dm + h * dh + c] = acc[c] * inv;
  }
  __syncthreads();
  if (tid < dm) {
    float m = 0.f;
    for (int p = 0; p < P; ++p) m += att[p * dm + tid];
    mean_att[tid] = m / float(P);
  }
  __syncthreads();
  if (tid < dm) {
    float v = bo[tid];
    for (int c = 0; c < dm; ++c) v = fmaf(mean_att[c], wo[tid * dm + c], v);
    pooled[size_t(s) * dm + tid] = v;
  }
}

// ---- the fused path: two kernels ---------------------------------------------------------------------------------
// k_cv_mlp runs the three per-pixel layers, k_cv_image everything after them with one work-group per image, the feature maps in LDS.
// Products run on the fp32 matrix cores (16x16x4; fp32 products and sums, like the scalar kernels above).  The weights are the FIRST operand:
// a result block is [channel][pixel] and a lane holds four neighbouring channels 4 lq .. 4 lq + 3 of pixel lr, which is one 16-byte
// access to a map with channels fastest.  The sum over k is order-free, so lane group lq takes the four consecutive k-values of unit
// 4 step + lq: one 16-byte read of either operand serves four matrix operations.
// Both kernels are bound by fetching their own code, which no cache holds when a launch begins: straight-line code costs about 2 us per
// KB (k_cv_mlp fully unrolled: 54 KB, 92 us; 21 KB: 46 us), so they are written as loops that run one copy of each piece.
typedef float f32x4_m __attribute__((ext_vector_type(4)));
typedef float f32x4_any __attribute__((ext_vector_type(4), aligned(4)));     // parameter vectors carry no alignment promise

struct CvBnArgs { const float *g, *o, *m, *v; };
struct CvMlpArgs {
  const uint16_t* x;                      // bf16 [M, cin]
  const float* w[3]; const float* b[3]; CvBnArgs bn[3];
  int n[3];
  float* out;                             // [M, n[2]]
  int M, cin;
};

// Layer 0: x is bf16 as it stands, and a weight of magnitude 2^-100 to 2^127 is the sum of three bf16 pieces exactly (bf16_pieces.h; a smaller one
// loses what lies below 2^-133), so three products on the bf16 matrix
// cores are the fp32 products, at a fifth of the time of the fp32 ones (16 x 16 x 32 in 48 cycles instead of 256).  The pieces are cut
// once per work-group on their way into LDS, in chunks of 256 channels (a single chunk stays for all tiles); sixteen waves share them,
// and a wave owns 16 pixels, whose values for 128 channels are requested ahead, past the end of a chunk too (started again with every chunk, 256
// images of 7 x 7 x 4096 took 106 us for layers of 16, 8 and 4, now 92; of 64, 8 and 4 134 and 118).  The later layers are fp32 products, weights in LDS too, and take the
// accumulators as they are: register r of block blk is channel 16 blk + 4 lq + r of pixel lr, i.e. the k-value of lane group lq.
// 256 images of 14 x 14 x 256: 30.6 us with the fp32 matrix cores and later layers' weights from memory, now 19.8 (a rolled loop of steps: 20.8
// unrolled by four).  Infinite or not representable operands leave NaN rests: a wave whose sums are not all finite takes them again from whole operands.
// Tiles of 16 pixels are dealt out over the work-groups wave by wave, so that each of 256 CUs gets 12 or 13 of the 3136 tiles of 256
// images of 14 x 14.
constexpr int MLP_KC = 256, MLP_ROWB = MLP_KC * 2 + 16;   // LDS bytes of a row of pieces: 16 rows start in 16 different bank quads
constexpr int MLP_ROW = CV_MAX_C + 4;                     // floats of a row of a later layer's weights
constexpr int MLP_PLANE = CV_MAX_C * MLP_ROWB;
constexpr int MLP_WAVES = 16;
typedef __bf16 bf16x8_m __attribute__((ext_vector_type(8)));
typedef uint32_t u32x4_m __attribute__((ext_vector_type(4)));
__global__ __launch_bounds__(MLP_WAVES * 64) void k_cv_mlp(const CvMlpArgs a) {
  __shared__ __align__(16) uint8_t wl[3 * MLP_PLANE];   // [piece][row][channel]
  __shared__ __align__(16) float wn[2][CV_MAX_C * MLP_ROW];
  __shared__ __align__(16) float pl[3][5][CV_MAX_C];    // per layer: bias, mean, 1 / sqrt(variance + eps), gain, offset
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, lr = lane & 15, lq = lane >> 4;
  const int tiles = (a.M + 15) / 16;
  const f32x4_m zero = {0.f, 0.f, 0.f, 0.f};
  const int nb0 = (a.n[0] + 15) / 16;
  if (tid < 3 * CV_MAX_C) {
    const int l = tid / CV_MAX_C, ch = tid % CV_MAX_C, c = min(ch, a.n[l] - 1);
    pl[l][0][ch] = a.b[l][c];
    pl[l][1][ch] = a.bn[l].m[c];
    pl[l][2][ch] = 1.0f / sqrtf(a.bn[l].v[c] + CV_BN_EPS);
    pl[l][3][ch] = a.bn[l].g[c];
    pl[l][4][ch] = a.bn[l].o[c];
  }
#pragma unroll 1
  for (int l = 0; l < 2; ++l)
#pragma unroll 1
    for (int i = tid; i < a.n[l + 1] * (a.n[l] / 4); i += MLP_WAVES * 64) {
      const int q = a.n[l] / 4, row = i / q, c = (i - row * q) * 4;
      *reinterpret_cast<f32x4_m*>(&wn[l][row * MLP_ROW + c]) = *reinterpret_cast<const f32x4_m*>(a.w[l + 1] + i * 4);
    }
#pragma unroll 1
  for (int t0 = 0; t0 < tiles; t0 += int(gridDim.x) * MLP_WAVES) {           // uniform over the work-group
    const int tile = t0 + wave * int(gridDim.x) + int(blockIdx.x);
    const bool live = tile < tiles;
    const int px = min(tile * 16 + lr, a.M - 1);
    const uint16_t* xr = a.x + size_t(px) * a.cin;
    f32x4_m h[4] = {zero, zero, zero, zero};
    auto load_x = [&](int c0) {                                              // eight channels of the lane's pixel; cin is a multiple of 4
      const int c = c0 + lq * 8;
      const uint2 u = c < a.cin ? *reinterpret_cast<const uint2*>(xr + c) : make_uint2(0u, 0u);
      const uint2 v = c + 4 < a.cin ? *reinterpret_cast<const uint2*>(xr + c + 4) : make_uint2(0u, 0u);
      return u32x4_m{u.x, u.y, v.x, v.y};
    };
    u32x4_m xb[4];                                                           // four steps ahead, across the chunks: on their way while weights are staged
#pragma unroll
    for (int j = 0; j < 4; ++j) xb[j] = load_x(j * 32);
#pragma unroll 1
    for (int kc = 0; kc < a.cin; kc += MLP_KC) {
      if (t0 == 0 || a.cin > MLP_KC) {
        __syncthreads();                                                     // the chunk before has been read
#pragma unroll 1
        for (int i = tid; i < a.n[0] * (MLP_KC / 8); i += MLP_WAVES * 64) {
          const int row = i / (MLP_KC / 8), c = (i % (MLP_KC / 8)) * 8;
          const float* p = a.w[0] + size_t(row) * a.cin + kc + c;
          const f32x4_m u = kc + c < a.cin ? *reinterpret_cast<const f32x4_m*>(p) : zero;
          const f32x4_m v = kc + c + 4 < a.cin ? *reinterpret_cast<const f32x4_m*>(p + 4) : zero;
          uint32_t o[3][4];
          cut3_pair(u.x, u.y, o[0][0], o[1][0], o[2][0]);
          cut3_pair(u.z, u.w, o[0][1], o[1][1], o[2][1]);
          cut3_pair(v.x, v.y, o[0][2], o[1][2], o[2][2]);
          cut3_pair(v.z, v.w, o[0][3], o[1][3], o[2][3]);
#pragma unroll
          for (int q = 0; q < 3; ++q)
            *reinterpret_cast<u32x4_m*>(wl + q * MLP_PLANE + row * MLP_ROWB + c * 2) = u32x4_m{o[q][0], o[q][1], o[q][2], o[q][3]};
        }
        __syncthreads();
      }
      if (!live) continue;
      const int steps = (min(MLP_KC, a.cin - kc) + 31) / 32;
#pragma unroll 1
      for (int st = 0; st < steps; ++st) {
        const bf16x8_m xv = __builtin_bit_cast(bf16x8_m, xb[0]);
        xb[0] = xb[1]; xb[1] = xb[2]; xb[2] = xb[3];
        xb[3] = load_x(kc + (st + 4) * 32);
#pragma unroll
        for (int b = 0; b < 4; ++b) {
          if (b < nb0) {                                                     // rows past n[0] repeat its last row: their results are never used
            const uint8_t* wr = wl + min(b * 16 + lr, a.n[0] - 1) * MLP_ROWB + st * 64 + lq * 16;
#pragma unroll
            for (int q = 2; q >= 0; --q)                                     // small terms first
              h[b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(*reinterpret_cast<const bf16x8_m*>(wr + q * MLP_PLANE), xv, h[b], 0, 0, 0);
          }
        }
      }
    }
    if (!live) continue;
    float check = 0.f;
#pragma unroll
    for (int b = 0; b < 4; ++b)
#pragma unroll
      for (int r = 0; r < 4; ++r) check = fmaf(h[b][r], 0.f, check);
    if (__ballot(check != check) != 0ull) {
#pragma unroll
      for (int b = 0; b < 4; ++b) h[b] = zero;
#pragma unroll 1
      for (int c = lq * 4; c < a.cin + lq * 4; c += 16) {                    // uniform trip count; channels past cin are zeros on both sides
        const uint2 xw = c < a.cin ? *reinterpret_cast<const uint2*>(xr + c) : make_uint2(0u, 0u);
        const float xv[4] = {__uint_as_float(xw.x << 16), __uint_as_float(xw.x & 0xffff0000u), __uint_as_float(xw.y << 16), __uint_as_float(xw.y & 0xffff0000u)};
#pragma unroll
        for (int b = 0; b < 4; ++b) {
          const f32x4_m wv = c < a.cin ? *reinterpret_cast<const f32x4_m*>(a.w[0] + size_t(min(b * 16 + lr, a.n[0] - 1)) * a.cin + c) : zero;
#pragma unroll
          for (int r = 0; r < 4; ++r) h[b] = __builtin_amdgcn_mfma_f32_16x16x4f32(wv[r], xv[r], h[b], 0, 0, 0);
        }
      }
    }
#pragma unroll 1
    for (int l = 0;; ++l) {
      // bias, batch norm, ReLU; channels that do not exist become 0
#pragma unroll
      for (int b = 0; b < 4; ++b) {
        const int c = b * 16 + 4 * lq;
        f32x4_m q[5];
#pragma unroll
        for (int j = 0; j < 5; ++j) q[j] = *reinterpret_cast<const f32x4_m*>(&pl[l][j][c]);
#pragma unroll
        for (int r = 0; r < 4; ++r) h[b][r] = c < a.n[l] ? fmaxf((h[b][r] + q[0][r] - q[1][r]) * q[2][r] * q[3][r] + q[4][r], 0.f) : 0.f;
      }
      if (l == 2) break;
      const int ni = a.n[l], no = a.n[l + 1];
      f32x4_m o[4] = {zero, zero, zero, zero};
#pragma unroll
      for (int b = 0; b < 4; ++b) {
        if (b * 16 < no) {
          const float* wr = &wn[l][min(b * 16 + lr, no - 1) * MLP_ROW];
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            if (i * 16 < ni) {                                               // uniform
              const int c = i * 16 + 4 * lq;
              const f32x4_m wv = c < ni ? *reinterpret_cast<const f32x4_m*>(wr + c) : zero;
#pragma unroll
              for (int r = 0; r < 4; ++r) o[b] = __builtin_amdgcn_mfma_f32_16x16x4f32(wv[r], h[i][r], o[b], 0, 0, 0);
            }
          }
        }
      }
#pragma unroll
      for (int b = 0; b < 4; ++b) h[b] = o[b];
    }
    if (tile * 16 + lr < a.M) {
#pragma unroll
      for (int b = 0; b < 4; ++b) {
        const int c = b * 16 + 4 * lq;
        if (c < a.n[2]) *reinterpret_cast<f32x4_m*>(a.out + size_t(px) * a.n[2] + c) = h[b];
      }
    }
  }
}

struct CvStageArgs {
  const float *wa, *wb, *ws;              // ws NULL: identity shortcut
  CvBnArgs bna, bnb, bns;
  const float *se1, *se1b, *se2, *se2b;
  int cin, cout, stride, hi, wi, ho, wo;
};
struct CvImageArgs {
  const float* in;                        // [S, h, w, c] output of the MLP
  CvStageArgs st[3];
  const float *wqkv, *bqkv, *wo, *bo, *w_out, *b_out;
  int heads, K;
  int32_t* idx;
  float* logits;
  int off_x, off_y, off_z;                // LDS offsets in floats: two padded maps, one plain map; the attention's arrays overlay x and z
};

constexpr int CV_THREADS = 1024, CV_WAVES = CV_THREADS / 64;
constexpr int CV_MAX_UNITS = 9 * CV_MAX_C / 4;
constexpr int CV_HEAD_FLOATS = CV_MAX_UNITS + 4 * CV_MAX_C + 16 * CV_MAX_C + MOQE_MAX_EXPERTS;     // tables at the start of the LDS
// Floats from one pixel to the next: an odd number of 16-byte units, so that 16 pixels start in 16 different bank quads.
__host__ __device__ inline int cv_pix(int c) { return (c / 4) % 2 ? c : c + 4; }

// The products of a work-group: a convolution, or a matrix product on the positions of a map.
enum CvOpKind { CV_OP_A, CV_OP_B, CV_OP_SHORT, CV_OP_QKV };
struct CvOp {
  const float* map; int row_step, col_step;   // source map and the floats between neighbouring output pixels' gathers
  const float* w; int units, cout;            // weights [cout][4 units]
  CvBnArgs bn;                                // CV_OP_QKV: o is the bias
  const float* inv_std;                       // LDS: 1 / sqrt(variance + eps) of each channel
  float* dst; int dst_row, dst_pix;           // result: dst + y * dst_row + x * dst_pix + channel
};

// a / b of numbers below 2^20 (a map has at most a few thousand pixels).  a + 1/2 is at least 1/2 away from every multiple of b, so the quotient at least
// 1 / (2 b) from a whole number; reciprocal (one ulp) and product (half of one) are off by less than 2^-22 of it, (a + 1/2) 2^-22 / b, which
// stays below that up to a = 2^21.
static __device__ __forceinline__ int cv_div(int a, int b) { return int((float(a) + 0.5f) * __builtin_amdgcn_rcpf(float(b))); }

// A wave's task is 16 pixels x 16 channels in steps of 16 k-values (four units; `delta` has entries up to a multiple of four).  A step's map
// values are read from LDS while the step before is multiplied, its weights are requested eight steps ahead through a buffer descriptor
// (a scalar offset per step: with addresses and clamps in vector instructions a step was as much vector as matrix work).  256 images
// of 14 x 14: k_cv_image 67.4 us with batches of four steps and a reciprocal square root per result, 64.4 with those once per product, now
// 61.  Sharing the steps of small maps out over idle waves was slower (72.8), the weights repacked to whole KiB no faster (66.0 + 1.7).
// Every lane of a result has channels co .. co + 3 of output pixel p.
static __device__ __forceinline__ void cv_products(const CvOp& op, CvOpKind kind, const int* delta, int P, int wo, const float* u, int upix, const float* gate) {
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(int(threadIdx.x) >> 6), lr = lane & 15, lq = lane >> 4;
  const int pbs = (P + 15) / 16, cbs = (op.cout + 15) / 16, units = op.units, steps = (units + 3) / 4;
  const bool partial = (units & 3) != 0;                                     // the last step has lanes without a unit
  const __amdgpu_buffer_rsrc_t w = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(op.w), 0, -1, 0x00020000);
  constexpr int NB = 8;
#pragma unroll 1
  for (int task = wave; task < pbs * cbs; task += CV_WAVES) {
    const int cb = cv_div(task, pbs), pb = task - cb * pbs;
    const int p = min(pb * 16 + lr, P - 1), y = cv_div(p, wo), x = p - y * wo;
    const float* src = op.map + y * op.row_step + x * op.col_step;
    const int co = cb * 16 + 4 * lq;                                         // cout is a multiple of 4: all four or none
    const int w_row = min(cb * 16 + lr, op.cout - 1) * units * 16;           // byte offset of the lane's weights, and in the last step
    const int w_any = w_row + lq * 16, w_last = w_row + (min(4 * (steps - 1) + lq, units - 1) - 4 * (steps - 1)) * 16;
    auto weights = [&](int st) {
      const int c = min(st, steps - 1);                                      // uniform
      return __builtin_bit_cast(f32x4_m, __builtin_amdgcn_raw_buffer_load_b128(w, c == steps - 1 ? w_last : w_any, c * 64, 0));
    };
    auto offset = [&](int st) { return delta[4 * min(st, steps - 1) + lq]; };
    f32x4_m wv[NB], av[2];
#pragma unroll
    for (int i = 0; i < NB; ++i) wv[i] = weights(i);
    av[0] = *reinterpret_cast<const f32x4_m*>(src + offset(0));
    int next = offset(1);
    const int cs = min(co, op.cout - 4);
    const f32x4_m qo = *reinterpret_cast<const f32x4_any*>(op.bn.o + cs);
    f32x4_m qg = {1.f, 1.f, 1.f, 1.f}, qm = {0.f, 0.f, 0.f, 0.f};
    if (kind != CV_OP_QKV) {
      qg = *reinterpret_cast<const f32x4_any*>(op.bn.g + cs);
      qm = *reinterpret_cast<const f32x4_any*>(op.bn.m + cs);
    }
    f32x4_m acc[2] = {{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}};
    auto step = [&](int st, int i) {                                         // i = st % NB
      av[(i + 1) & 1] = *reinterpret_cast<const f32x4_m*>(src + next);
      next = offset(st + 2);
      if (partial && st == steps - 1) {                                      // units past the end are zeros on both sides
        const bool in = 4 * st + lq < units;
#pragma unroll
        for (int r = 0; r < 4; ++r) { wv[i][r] = in ? wv[i][r] : 0.f; av[i & 1][r] = in ? av[i & 1][r] : 0.f; }
      }
#pragma unroll
      for (int r = 0; r < 4; ++r) acc[r & 1] = __builtin_amdgcn_mfma_f32_16x16x4f32(wv[i][r], av[i & 1][r], acc[r & 1], 0, 0, 0);
    };
    // Whole rounds of the ring carry no branch around a request: with one, a wait has to allow for the request not having been made, and
    // waits for the latest instead of the oldest.
    int s = 0;
#pragma unroll 1
    for (; s + NB <= steps; s += NB) {
#pragma unroll
      for (int i = 0; i < NB; ++i) {
        step(s + i, i);
        wv[i] = weights(s + i + NB);
      }
    }
#pragma unroll
    for (int i = 0; i < NB - 1; ++i)
      if (s + i < steps) step(s + i, i);                                     // uniform
    f32x4_m v = acc[0] + acc[1];
    if (pb * 16 + lr < P && co < op.cout) {
      if (kind == CV_OP_QKV) v = v + qo;
      else {
        const f32x4_m qi = *reinterpret_cast<const f32x4_m*>(op.inv_std + cs);
#pragma unroll
        for (int r = 0; r < 4; ++r) v[r] = (v[r] - qm[r]) * qi[r] * qg[r] + qo[r];
      }
      if (kind == CV_OP_SHORT) {                                             // the stage's result: relu(u * gate + shortcut)
#pragma unroll
        for (int r = 0; r < 4; ++r) v[r] = fmaf(u[p * upix + co + r], gate[co + r], v[r]);
      }
      if (kind == CV_OP_A || kind == CV_OP_SHORT) {
#pragma unroll
        for (int r = 0; r < 4; ++r) v[r] = fmaxf(v[r], 0.f);
      }
      *reinterpret_cast<f32x4_m*>(op.dst + y * op.dst_row + x * op.dst_pix + co) = v;
    }
  }
}

// One work-group per image: the three stages (both convolutions, excitation, shortcut), attention over the last map, logits, arg-max.
// The maps stay in LDS with a border of zeros, so the 3x3 gather needs no bounds.
__global__ __launch_bounds__(CV_THREADS) void k_cv_image(const CvImageArgs a) {
  extern __shared__ __align__(16) float lds[];
  int* delta = reinterpret_cast<int*>(lds);                                  // [CV_MAX_UNITS] map offset of each unit of four k-values
  float* gate = lds + CV_MAX_UNITS;                                          // [64]
  float* mean = gate + CV_MAX_C;                                             // [64]
  float* hid = mean + CV_MAX_C;                                              // [64]
  float* pooled = hid + CV_MAX_C;                                            // [64]
  float* inv_std = pooled;                                                   // until the last product: the pooled row comes later
  float* part = pooled + CV_MAX_C;                                           // [16][64]
  float* zl = part + 16 * CV_MAX_C;                                          // [experts]
  const int tid = threadIdx.x, s = blockIdx.x;
  float *cur = lds + a.off_x, *oth = lds + a.off_y, *u = lds + a.off_z;
  {
    const int c = a.st[0].cin, c4 = c / 4, hi = a.st[0].hi, wi = a.st[0].wi, pix = cv_pix(c), W = wi + 2;
#pragma unroll 1
    for (int i = tid; i < (hi + 2) * W * pix; i += CV_THREADS) cur[i] = 0.f;
    __syncthreads();
    const float* src = a.in + size_t(s) * hi * wi * c;
#pragma unroll 1
    for (int i = tid; i < hi * wi * c4; i += CV_THREADS) {
      const int p = i / c4, k = (i - p * c4) * 4, y = p / wi, x = p - y * wi;
      *reinterpret_cast<f32x4_m*>(cur + ((y + 1) * W + x + 1) * pix + k) = *reinterpret_cast<const f32x4_m*>(src + size_t(p) * c + k);
    }
  }
  // ten products: two convolutions and the shortcut of each stage, then queries, keys and values
  const int dm = a.st[2].cout, P3 = a.st[2].ho * a.st[2].wo, row = 3 * dm + 4;
  float* qkv = lds + a.off_x;                                                // [P][3 dm + 4]
  // The reciprocal square root of a product's variances is some sixty instructions per channel: taken once per product, by a wave that has
  // little else to do, with the variances requested a product ahead.
  const int ic = tid - (CV_THREADS - 64);
  auto variance = [&](int n) {
    const CvStageArgs& t = a.st[min(n / 3, 2)];
    const float* v = n % 3 == 0 ? t.bna.v : n % 3 == 1 ? t.bnb.v : t.bns.v;
    return ic >= 0 && n < 9 && (n % 3 < 2 || t.ws) ? v[min(ic, t.cout - 1)] : 0.f;
  };
  float var = variance(0);
#pragma unroll 1
  for (int n = 0; n < 10; ++n) {
    if (ic >= 0) inv_std[ic] = 1.0f / sqrtf(var + CV_BN_EPS);
    var = variance(n + 1);
    const CvStageArgs& t = a.st[n == 9 ? 2 : n / 3];
    const CvOpKind kind = n == 9 ? CV_OP_QKV : CvOpKind(n % 3);
    const int pi = cv_pix(t.cin), po = cv_pix(t.cout), Wi = t.wi + 2, Wo = t.wo + 2, P = t.ho * t.wo;
    const bool from_a = kind == CV_OP_B || kind == CV_OP_QKV;                // gathers from a map of the stage's output size
    const int gc = from_a ? t.cout : t.cin, gW = from_a ? Wo : Wi, gp = from_a ? po : pi, taps = kind == CV_OP_A || kind == CV_OP_B ? 9 : 1;
    CvOp op;
    op.map = kind == CV_OP_B ? oth : cur;
    op.units = taps * gc / 4;
    const int step = kind == CV_OP_A || kind == CV_OP_SHORT ? t.stride : 1;
    op.row_step = step * gW * gp; op.col_step = step * gp;
    op.cout = kind == CV_OP_QKV ? 3 * dm : t.cout;
    op.w = kind == CV_OP_A ? t.wa : kind == CV_OP_B ? t.wb : kind == CV_OP_SHORT ? t.ws : a.wqkv;
    op.bn = kind == CV_OP_A ? t.bna : kind == CV_OP_B ? t.bnb : kind == CV_OP_SHORT ? t.bns : CvBnArgs{nullptr, a.bqkv, nullptr, nullptr};
    op.inv_std = inv_std;
    op.dst = oth + (Wo + 1) * po; op.dst_row = Wo * po; op.dst_pix = po;
    if (kind == CV_OP_B) { op.dst = u; op.dst_row = t.wo * po; }
    if (kind == CV_OP_QKV) { op.dst = qkv; op.dst_row = t.wo * row; op.dst_pix = row; }
    if (kind == CV_OP_A) {
#pragma unroll 1
      for (int j = tid; j < (t.ho + 2) * Wo * po; j += CV_THREADS) oth[j] = 0.f;
    }
    if (tid < (op.units + 3) / 4 * 4) {                                      // entries past the end repeat the last
      const int un = min(tid, op.units - 1), tap = 4 * un / gc, c = 4 * un - tap * gc;
      delta[tid] = taps == 9 ? ((tap / 3) * gW + tap % 3) * gp + c : (gW + 1) * gp + c;
    }
    if (kind == CV_OP_SHORT) {
      // excitation: channel means of u, two small layers, sigmoid
      const int Cr = t.cout / 4, c = tid & 63, q = tid >> 6;
      float acc = 0.f;
      if (c < t.cout) {
#pragma unroll 2
        for (int p = q; p < P; p += 16) acc += u[p * po + c];
      }
      part[q * CV_MAX_C + c] = acc;
      __syncthreads();
      if (tid < t.cout) {
        float v = part[tid];
#pragma unroll 3
        for (int k = 1; k < 16; ++k) v += part[k * CV_MAX_C + tid];
        mean[tid] = v / float(P);
      }
      __syncthreads();
      if (tid < 16 * Cr) {                                                   // 16 lanes per hidden unit
        const int h = tid >> 4;
        float v = 0.f;
#pragma unroll 2
        for (int k = tid & 15; k < t.cout; k += 16) v = fmaf(t.se1[h * t.cout + k], mean[k], v);
#pragma unroll
        for (int d = 8; d >= 1; d >>= 1) v += __shfl_xor(v, d);
        if ((tid & 15) == 0) hid[h] = fmaxf(v + t.se1b[h], 0.f);
      }
      __syncthreads();
      if (tid < t.cout) {
        float g = t.se2b[tid];
#pragma unroll 4
        for (int k = 0; k < Cr; ++k) g = fmaf(t.se2[tid * Cr + k], hid[k], g);
        gate[tid] = 1.0f / (1.0f + expf(-g));
      }
    }
    __syncthreads();
    if (kind != CV_OP_SHORT || t.ws) {
      cv_products(op, kind, delta, P, t.wo, u, po, gate);
    } else {                                                                 // identity (stride 1, equal widths): the maps coincide
#pragma unroll 1
      for (int j = tid; j < P * t.cout; j += CV_THREADS) {
        const int p = j / t.cout, c = j - p * t.cout, y = p / t.wo, x = p - y * t.wo, at = ((y + 1) * Wo + x + 1) * po + c;
        oth[at] = fmaxf(fmaf(u[p * po + c], gate[c], cur[at]), 0.f);
      }
    }
    __syncthreads();
    if (kind == CV_OP_SHORT) { float* tmp = cur; cur = oth; oth = tmp; }     // the next map, in the buffer of a; its border is still zero
  }
  // Attention over the P positions.  Only the mean over the queries is needed: mean_q sum_k p[q][k] v[k] = sum_k (mean_q p[q][k]) v[k].
  const int P = P3, dh = dm / a.heads;
  float* sc = qkv + P * row;                                                 // [heads][P queries][P keys]
  const float scale = 1.0f / sqrtf(float(dh));
#pragma unroll 1
  for (int j = tid; j < a.heads * P * P; j += CV_THREADS) {
    const int k = j % P, q = (j / P) % P, h = j / (P * P);
    const float *qv = qkv + q * row + h * dh, *kv = qkv + k * row + dm + h * dh;
    float d = 0.f;
#pragma unroll 4
    for (int c = 0; c < dh; ++c) d = fmaf(qv[c], kv[c], d);
    sc[j] = d * scale;
  }
  __syncthreads();
#pragma unroll 1
  for (int r0 = 0; r0 < a.heads * P; r0 += CV_THREADS / 8) {                 // eight lanes per row of scores
    const int r = r0 + (tid >> 3);
    if (r < a.heads * P) {
      float* v = sc + r * P;
      float mx = -INFINITY, sum = 0.f;
#pragma unroll 2
      for (int k = tid & 7; k < P; k += 8) mx = fmaxf(mx, v[k]);
#pragma unroll
      for (int d = 4; d >= 1; d >>= 1) mx = fmaxf(mx, __shfl_xor(mx, d));
#pragma unroll 1
      for (int k = tid & 7; k < P; k += 8) { const float e = expf(v[k] - mx); v[k] = e; sum += e; }
#pragma unroll
      for (int d = 4; d >= 1; d >>= 1) sum += __shfl_xor(sum, d);
      const float inv = 1.0f / sum;
#pragma unroll 1
      for (int k = tid & 7; k < P; k += 8) v[k] *= inv;
    }
  }
  __syncthreads();
#pragma unroll 1
  for (int j = tid; j < a.heads * P; j += CV_THREADS) {
    const int k = j % P, h = j / P;
    float m = 0.f;
#pragma unroll 4
    for (int q = 0; q < P; ++q) m += sc[(h * P + q) * P + k];
    qkv[k * row + h] = m / float(P);                                         // queries are no longer needed: heads <= dm
  }
  __syncthreads();
  if (tid < dm) {
    const int h = tid / dh;
    float m = 0.f;
#pragma unroll 4
    for (int k = 0; k < P; ++k) m = fmaf(qkv[k * row + h], qkv[k * row + 2 * dm + tid], m);
    mean[tid] = m;
  }
  __syncthreads();
  // output projection, then the logits: 16 lanes per output
#pragma unroll 1
  for (int l = 0; l < 2; ++l) {
    const int j = tid >> 4, n = l ? a.K : dm;
    const float *w = l ? a.w_out : a.wo, *b = l ? a.b_out : a.bo, *in = l ? pooled : mean;
    if (j < n) {
      float v = 0.f;
#pragma unroll 4
      for (int c = tid & 15; c < dm; c += 16) v = fmaf(in[c], w[j * dm + c], v);
#pragma unroll
      for (int d = 8; d >= 1; d >>= 1) v += __shfl_xor(v, d);
      if ((tid & 15) == 0) {
        if (b) v += b[j];
        (l ? zl : pooled)[j] = v;
        if (l && a.logits) a.logits[size_t(s) * a.K + j] = v;
      }
    }
    __syncthreads();
  }
  if (tid == 0) {
    float best = zl[0];
    int best_k = 0;
#pragma unroll 1
    for (int k = 1; k < a.K; ++k)
      if (zl[k] > best) { best = zl[k]; best_k = k; }                        // strict >: ties keep the lowest index
    a.idx[s] = best_k;
  }
}

// ---- host side -------------------------------------------------------------------------------------------------
namespace {
int out_size(int n, int taps, int stride) { return taps == 9 ? (n + 2 - 3) / stride + 1 : (n - 1) / stride + 1; }

struct CvLayout {
  size_t buf[4], gate, pooled, head, total;
  int h[4], w[4];            // feature-map size entering stage 0, 1, 2 and leaving stage 2
};

CvLayout cv_layout(int S, int h, int w, const moqe_cv_router& r) {
  CvLayout L;
  L.h[0] = h; L.w[0] = w;
  for (int i = 0; i < 3; ++i) {
    L.h[i + 1] = out_size(L.h[i], 9, r.stage[i].stride);
    L.w[i + 1] = out_size(L.w[i], 9, r.stage[i].stride);
  }
  size_t o = 0;
  const size_t big = align256(size_t(S) * h * w * CV_MAX_C * 4);        // any feature map fits
  for (int i = 0; i < 4; ++i) { L.buf[i] = o; o += big; }
  L.gate = o;   o += align256(size_t(S) * CV_MAX_C * 4);
  L.pooled = o; o += align256(size_t(S) * CV_MAX_C * 4);
  moqe_router head{nullptr, nullptr, r.w_out, r.b_out, r.stage[2].cout, 0, r.n_experts};
  L.head = o;   o += align256(route_ws_bytes(S, 1, head));
  L.total = o;
  return L;
}

int32_t conv(const void* in, bool in_bf16, const float* w, const float* bias, const moqe_bn* bn, float* out, int S, int hi, int wi, int cin,
             int cout, int taps, int stride, bool relu, hipStream_t st) {
  CvConvArgs a;
  memset(&a, 0, sizeof(a));
  a.in = in; a.in_bf16 = in_bf16 ? 1 : 0; a.w = w; a.bias = bias; a.out = out;
  if (bn) { a.bn_g = bn->gain; a.bn_o = bn->offset; a.bn_m = bn->mean; a.bn_v = bn->var; }
  a.S = S; a.hi = hi; a.wi = wi; a.cin = cin; a.cout = cout; a.taps = taps; a.stride = stride; a.relu = relu ? 1 : 0;
  a.ho = out_size(hi, taps, stride); a.wo = out_size(wi, taps, stride);
  const long M = long(S) * a.ho * a.wo;
  ProfileScope ps(MOQE_PK_ROUTE, st);
  if (cout <= 16) hipLaunchKernelGGL(k_cv_conv<16>, dim3(unsigned((M + 255) / 256), (cout + 15) / 16), dim3(256), 0, st, a);
  else if (cout <= 32) hipLaunchKernelGGL(k_cv_conv<32>, dim3(unsigned((M + 127) / 128), (cout + 31) / 32), dim3(256), 0, st, a);
  else hipLaunchKernelGGL(k_cv_conv<64>, dim3(unsigned((M + 63) / 64), (cout + 63) / 64), dim3(256), 0, st, a);
  return check_launch("route_cv(convolution)");
}

// LDS of the fused path for this router and image size, in floats; fills the buffer offsets.
size_t cv_image_lds(const CvLayout& L, const moqe_cv_router& r, int* off_x, int* off_y, int* off_z) {
  size_t x = 0, y = 0, z = 0;
  int cin = r.mlp_n[2];
  for (int i = 0; i < 3; ++i) {
    const int cout = r.stage[i].cout;
    size_t& in = i % 2 ? y : x;                       // the maps alternate between two buffers
    size_t& out = i % 2 ? x : y;
    in = std::max(in, size_t(L.h[i] + 2) * (L.w[i] + 2) * cv_pix(cin));
    out = std::max(out, size_t(L.h[i + 1] + 2) * (L.w[i + 1] + 2) * cv_pix(cout));
    z = std::max(z, size_t(L.h[i + 1]) * L.w[i + 1] * cv_pix(cout));
    cin = cout;
  }
  const size_t P = size_t(L.h[3]) * L.w[3], qkv = P * (3 * cin + 4) + size_t(r.n_heads) * P * P;
  x = std::max(x, qkv > z ? qkv - z : 0);             // x and z lie side by side and hold the attention's arrays at the end
  x = (x + 3) / 4 * 4; y = (y + 3) / 4 * 4;
  const size_t head = (CV_HEAD_FLOATS + 3) / 4 * 4;
  *off_y = int(head); *off_x = int(head + y); *off_z = int(head + y + x);
  return head + y + x + z;
}

bool bn_ok(const moqe_bn& b) { return b.gain && b.offset && b.mean && b.var; }
}  // namespace

int32_t check_cv_router(const moqe_cv_router* r, int h, int w, const char* who) {
  if (!r) return set_error(MOQE_E_NULL, "%s: router is NULL", who);
  if (r->n_experts < 1 || r->n_experts > MOQE_MAX_EXPERTS) return set_error(MOQE_E_SHAPE, "%s: n_experts=%d", who, r->n_experts);
  if (r->c_in <= 0 || r->c_in % 4 || h <= 0 || w <= 0)
    return set_error(MOQE_E_SHAPE, "%s: image %d x %d x %d (channels a multiple of 4)", who, h, w, r->c_in);
  for (int i = 0; i < 3; ++i) {
    if (!r->mlp_w[i] || !r->mlp_b[i] || !bn_ok(r->mlp_bn[i])) return set_error(MOQE_E_NULL, "%s: MLP layer %d has a NULL parameter", who, i);
    if (r->mlp_n[i] <= 0 || r->mlp_n[i] > CV_MAX_C || r->mlp_n[i] % 4)
      return set_error(MOQE_E_SHAPE, "%s: MLP width %d must be a multiple of 4, at most %d", who, r->mlp_n[i], CV_MAX_C);
    const moqe_cv_stage& s = r->stage[i];
    const int cin = i == 0 ? r->mlp_n[2] : r->stage[i - 1].cout;
    if (!s.conv_a || !s.conv_b || !bn_ok(s.bn_a) || !bn_ok(s.bn_b) || !s.se_w1 || !s.se_b1 || !s.se_w2 || !s.se_b2)
      return set_error(MOQE_E_NULL, "%s: stage %d has a NULL parameter", who, i);
    if (s.cout <= 0 || s.cout > CV_MAX_C || s.cout % 4 || (s.stride != 1 && s.stride != 2))
      return set_error(MOQE_E_SHAPE, "%s: stage %d: %d channels (multiple of 4, at most %d), stride %d (1 or 2)", who, i, s.cout, CV_MAX_C, s.stride);
    if (!s.short_w && (s.stride != 1 || s.cout != cin))
      return set_error(MOQE_E_SHAPE, "%s: stage %d changes stride or width and needs a shortcut convolution", who, i);
    if (s.short_w && !bn_ok(s.short_bn)) return set_error(MOQE_E_NULL, "%s: stage %d: the shortcut's batch norm is NULL", who, i);
  }
  if (!r->wqkv || !r->bqkv || !r->wo || !r->bo || !r->w_out) return set_error(MOQE_E_NULL, "%s: an attention or output parameter is NULL", who);
  for (int i = 0; i < 3; ++i) {
    const void* mats[] = {r->mlp_w[i], r->stage[i].conv_a, r->stage[i].conv_b, r->stage[i].short_w};
    for (const void* m : mats)
      if (reinterpret_cast<uintptr_t>(m) % 16) return set_error(MOQE_E_SHAPE, "%s: weight matrices and filters must be 16-byte aligned", who);
  }
  const int dm = r->stage[2].cout;
  if (r->n_heads <= 0 || dm % r->n_heads || dm / r->n_heads > CV_MAX_DH || dm % 8)
    return set_error(MOQE_E_SHAPE, "%s: %d heads on %d channels (head width at most %d, channels a multiple of 8)", who, r->n_heads, dm, CV_MAX_DH);
  if (reinterpret_cast<uintptr_t>(r->w_out) % 16) return set_error(MOQE_E_SHAPE, "%s: w_out must be 16-byte aligned", who);
  int hh = h, ww = w;
  for (int i = 0; i < 3; ++i) { hh = out_size(hh, 9, r->stage[i].stride); ww = out_size(ww, 9, r->stage[i].stride); }
  if (hh * ww > CV_MAX_POS) return set_error(MOQE_E_SHAPE, "%s: the last feature map has %d positions, at most %d", who, hh * ww, CV_MAX_POS);
  return MOQE_OK;
}

size_t route_cv_ws_bytes(int S, int h, int w, const moqe_cv_router& r) { return cv_layout(S, h, w, r).total; }

int32_t launch_route_cv(const void* x, int S, int h, int w, const moqe_cv_router& r, int32_t* idx, float* logits, void* ws, hipStream_t st) {
  const CvLayout L = cv_layout(S, h, w, r);
  uint8_t* p = static_cast<uint8_t*>(ws);
  float* buf[4];
  for (int i = 0; i < 4; ++i) buf[i] = reinterpret_cast<float*>(p + L.buf[i]);
  float* gate = reinterpret_cast<float*>(p + L.gate);
  float* pooled = reinterpret_cast<float*>(p + L.pooled);
  int32_t rc;
  // The fused path keeps an image's maps in LDS: the paper's channels fit up to 24 x 24.  What does not fit takes the kernels below, one
  // launch per layer.
  CvImageArgs ia;
  memset(&ia, 0, sizeof(ia));
  const size_t lds = cv_image_lds(L, r, &ia.off_x, &ia.off_y, &ia.off_z) * 4;
  if (lds <= size_t(CV_LDS_MAX)) {
    if ((rc = ensure_dynamic_lds(LDSK_CV_IMAGE, reinterpret_cast<const void*>(&k_cv_image), CV_LDS_MAX, "route_cv"))) return rc;
    auto bn = [](const moqe_bn& b) { return CvBnArgs{b.gain, b.offset, b.mean, b.var}; };
    CvMlpArgs ma;
    memset(&ma, 0, sizeof(ma));
    ma.x = static_cast<const uint16_t*>(x);
    for (int i = 0; i < 3; ++i) { ma.w[i] = r.mlp_w[i]; ma.b[i] = r.mlp_b[i]; ma.bn[i] = bn(r.mlp_bn[i]); ma.n[i] = r.mlp_n[i]; }
    ma.out = buf[0]; ma.M = S * h * w; ma.cin = r.c_in;
    ia.in = buf[0];
    int cin = r.mlp_n[2];
    for (int i = 0; i < 3; ++i) {
      const moqe_cv_stage& sg = r.stage[i];
      ia.st[i] = CvStageArgs{sg.conv_a, sg.conv_b, sg.short_w, bn(sg.bn_a), bn(sg.bn_b), bn(sg.short_bn), sg.se_w1, sg.se_b1, sg.se_w2, sg.se_b2,
                             cin, sg.cout, sg.stride, L.h[i], L.w[i], L.h[i + 1], L.w[i + 1]};
      cin = sg.cout;
    }
    ia.wqkv = r.wqkv; ia.bqkv = r.bqkv; ia.wo = r.wo; ia.bo = r.bo; ia.w_out = r.w_out; ia.b_out = r.b_out;
    ia.heads = r.n_heads; ia.K = r.n_experts; ia.idx = idx; ia.logits = logits;
    const int tiles = (ma.M + 15) / 16;
    ProfileScope ps(MOQE_PK_ROUTE, st);
    hipLaunchKernelGGL(k_cv_mlp, dim3(std::min(tiles, 256)), dim3(MLP_WAVES * 64), 0, st, ma);
    hipLaunchKernelGGL(k_cv_image, dim3(S), dim3(CV_THREADS), lds, st, ia);
    return check_launch("route_cv(fused)");
  }
  // per-pixel MLP: x -> buf0 -> buf1 -> buf0
  if ((rc = conv(x, true, r.mlp_w[0], r.mlp_b[0], &r.mlp_bn[0], buf[0], S, h, w, r.c_in, r.mlp_n[0], 1, 1, true, st))) return rc;
  if ((rc = conv(buf[0], false, r.mlp_w[1], r.mlp_b[1], &r.mlp_bn[1], buf[1], S, h, w, r.mlp_n[0], r.mlp_n[1], 1, 1, true, st))) return rc;
  if ((rc = conv(buf[1], false, r.mlp_w[2], r.mlp_b[2], &r.mlp_bn[2], buf[0], S, h, w, r.mlp_n[1], r.mlp_n[2], 1, 1, true, st))) return rc;
  float* cur = buf[0];                      // the stage's input
  int cin = r.mlp_n[2];
  for (int i = 0; i < 3; ++i) {
    const moqe_cv_stage& sg = r.stage[i];
    float* free_buf[3];
    int nf = 0;
    for (int b = 0; b < 4; ++b)
      if (buf[b] != cur) free_buf[nf++] = buf[b];
    float *a = free_buf[0], *u = free_buf[1], *sc = free_buf[2];
    const int hi = L.h[i], wi = L.w[i], ho = L.h[i + 1], wo = L.w[i + 1], P = ho * wo;
    if ((rc = conv(cur, false, sg.conv_a, nullptr, &sg.bn_a, a, S, hi, wi, cin, sg.cout, 9, sg.stride, true, st))) return rc;
    if ((rc = conv(a, false, sg.conv_b, nullptr, &sg.bn_b, u, S, ho, wo, sg.cout, sg.cout, 9, 1, false, st))) return rc;
    const float* shortcut = cur;
    if (sg.short_w) {
      if ((rc = conv(cur, false, sg.short_w, nullptr, &sg.short_bn, sc, S, hi, wi, cin, sg.cout, 1, sg.stride, false, st))) return rc;
      shortcut = sc;
    }
    {
      ProfileScope ps(MOQE_PK_ROUTE, st);
      hipLaunchKernelGGL(k_cv_se_gate, dim3(S), dim3(256), 0, st, u, P, sg.cout, sg.se_w1, sg.se_b1, sg.se_w2, sg.se_b2, gate);
      const size_t total = size_t(S) * P * sg.cout;
      hipLaunchKernelGGL(k_cv_se_apply, dim3(unsigned((total + 255) / 256)), dim3(256), 0, st, u, gate, shortcut, a, S, P, sg.cout);
      if ((rc = check_launch("route_cv(squeeze and excitation)"))) return rc;
    }
    cur = a;                                 // a is free again once u has been computed from it
    cin = sg.cout;
  }
  const int P = L.h[3] * L.w[3], dm = cin;
  {
    ProfileScope ps(MOQE_PK_ROUTE, st);
    const size_t lds = size_t(P) * 5 * dm * 4 + size_t(dm) * 4;
    hipLaunchKernelGGL(k_cv_attn_pool, dim3(S), dim3(256), lds, st, cur, P, dm, r.n_heads, r.wqkv, r.bqkv, r.wo, r.bo, pooled);
    if ((rc = check_launch("route_cv(attention)"))) return rc;
  }
  moqe_router head{nullptr, nullptr, r.w_out, r.b_out, dm, 0, r.n_experts};
  return launch_route_features(pooled, S, head, idx, logits, p + L.head, st);
}

}  // namespace moqe
