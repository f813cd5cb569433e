// Router: mean pooling, [Linear -> ReLU ->] Linear, top-1 selection (MoQE Section 3.2: the
// router is a classifier whose last stage is an MLP producing one logit per expert; one
// expert is activated per sample, Section 3.1).  All reductions run in a fixed order, so
// results are bit-reproducible from launch to launch.
#include "bucket_device.h"

namespace moqe {

static __device__ __forceinline__ float bf16_bits_to_float(uint32_t b) { return __uint_as_float(b << 16); }

static __device__ __forceinline__ float wave_sum(float v) {
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) v += __shfl_xor(v, off, 64);
  return v;
}

// partial[s][c][d] = sum over the tokens of chunk c of x[s][t][d].
// Block: 256 threads = CT column-threads (8 columns each) x TR token-rows.
// With one chunk (C == 1, `finish` set) the sum is divided by T here and written as the pooled feature: the
// arithmetic of k_pool_finish on a single chunk (0 + sum, then the division), without its launch.
__global__ __launch_bounds__(256) void k_pool_partial(const uint16_t* __restrict__ x, float* __restrict__ partial,
                                                       int T, int D, int C, int CT, int finish) {
  __shared__ float red[256 * 8];
  const int s = blockIdx.z, c = blockIdx.y;
  const int TR = 256 / CT;
  const int ct = threadIdx.x % CT, tr = threadIdx.x / CT;
  const int col = (blockIdx.x * CT + ct) * 8;
  const int tchunk = (T + C - 1) / C;
  const int t0 = c * tchunk, t1 = min(T, t0 + tchunk);
  float acc[8];
#pragma unroll
  for (int i = 0; i < 8; ++i) acc[i] = 0.f;
  if (col < D) {
    const uint16_t* base = x + (size_t(s) * T) * D + col;
    // eight rows' loads in flight (rows past the chunk's end are clamped, loaded and not added); the additions keep
    // their order
    for (int t = t0 + tr; t < t1; t += 8 * TR) {
      uint4 v4[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) v4[u] = *reinterpret_cast<const uint4*>(base + size_t(min(t + u * TR, t1 - 1)) * D);
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        if (t + u * TR < t1) {
          const uint4 v = v4[u];
          acc[0] += bf16_bits_to_float(v.x & 0xffffu); acc[1] += bf16_bits_to_float(v.x >> 16);
          acc[2] += bf16_bits_to_float(v.y & 0xffffu); acc[3] += bf16_bits_to_float(v.y >> 16);
          acc[4] += bf16_bits_to_float(v.z & 0xffffu); acc[5] += bf16_bits_to_float(v.z >> 16);
          acc[6] += bf16_bits_to_float(v.w & 0xffffu); acc[7] += bf16_bits_to_float(v.w >> 16);
        }
      }
    }
  }
#pragma unroll
  for (int i = 0; i < 8; ++i) red[threadIdx.x * 8 + i] = acc[i];
  __syncthreads();
  if (tr == 0 && col < D) {
    float* out = partial + (size_t(s) * C + c) * D + col;
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      float v = 0.f;
      for (int r = 0; r < TR; ++r) v += red[(r * CT + ct) * 8 + i];   // fixed order
      out[i] = finish ? __fdiv_rn(v, float(T)) : v;
    }
  }
}

// pooled[s][d] = (sum_c partial[s][c][d]) / T
__global__ void k_pool_finish(const float* __restrict__ partial, float* __restrict__ pooled, int S, int T, int D, int C) {
  size_t i = size_t(blockIdx.x) * blockDim.x + threadIdx.x;
  if (i >= size_t(S) * D) return;
  int s = int(i / D), d = int(i % D);
  float v = 0.f;
  for (int c = 0; c < C; ++c) v += partial[(size_t(s) * C + c) * D + d];
  pooled[i] = __fdiv_rn(v, float(T));
}

// Hidden layer on the fp32 matrix cores.  part[kz][s][j] = sum over k-slice kz of feat[s][k] * w1[j][k]
// for one tile of 16 samples x 16 hidden units.  The tile's operands are first copied to LDS with
// coalesced loads (one round trip: every load of the work-group is issued before any is used; a
// direct operand-shaped read touches 64 cache lines per instruction and is bound by the texture
// path), then each of the 4 waves multiplies a quarter of the slice and the four partial tiles
// are added through LDS in wave order.  Bias and ReLU are applied by the consumer, which adds the
// slices in order, so the result does not depend on scheduling.
// XBF16: feat is the bf16 activation matrix itself (T == 1, pooling is the identity).
typedef float f32x4_t __attribute__((ext_vector_type(4)));
static __device__ __forceinline__ float4 keep4(float4 v, bool ok) {
  return make_float4(ok ? v.x : 0.f, ok ? v.y : 0.f, ok ? v.z : 0.f, ok ? v.w : 0.f);
}
constexpr int HID_KC = 512;                       // columns per k-slice
constexpr int HID_STRIDE = HID_KC + 4;            // LDS row stride in floats (bank-conflict free b128 reads)

template <bool XBF16>
__global__ __launch_bounds__(256) void k_router_hidden(const void* __restrict__ feat, const float* __restrict__ w1,
                                                        float* __restrict__ part, int S, int D, int Hd) {
  __shared__ __align__(16) float wt[16 * HID_STRIDE];
  __shared__ __align__(16) float xt[16 * HID_STRIDE];
  __shared__ float red[3][4][64];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int h0 = blockIdx.x * 16, s0 = blockIdx.y * 16, kz = blockIdx.z;
  const int kbeg = kz * HID_KC;
  // ---- stage: thread t copies columns 4*(t%128) .. +3 of rows t/128, t/128 + 2, ... ----
  {
    const int c4 = (tid & 127) * 4;
    const bool kin = kbeg + c4 < D;
    const int kc = kin ? kbeg + c4 : 0;
#pragma unroll
    for (int r = 0; r < 8; ++r) {
      const int row = (tid >> 7) + 2 * r;
      const int hr = min(h0 + row, Hd - 1), sr = min(s0 + row, S - 1);
      const float4 wv = *reinterpret_cast<const float4*>(w1 + size_t(hr) * D + kc);
      float4 xv;
      if constexpr (XBF16) {
        const uint2 v = *reinterpret_cast<const uint2*>(static_cast<const uint16_t*>(feat) + size_t(sr) * D + kc);
        xv = make_float4(__uint_as_float(v.x << 16), __uint_as_float(v.x & 0xffff0000u),
                         __uint_as_float(v.y << 16), __uint_as_float(v.y & 0xffff0000u));
      } else {
        xv = *reinterpret_cast<const float4*>(static_cast<const float*>(feat) + size_t(sr) * D + kc);
      }
      const bool wok = kin && h0 + row < Hd, xok = kin && s0 + row < S;
      *reinterpret_cast<float4*>(wt + row * HID_STRIDE + c4) = keep4(wv, wok);
      *reinterpret_cast<float4*>(xt + row * HID_STRIDE + c4) = keep4(xv, xok);
    }
  }
  __syncthreads();
  // ---- multiply: wave w takes columns [128w, 128w + 128): 8 steps of 16 columns ----
  const int i = lane & 15, q = lane >> 4;
  f32x4_t acc0 = {0.f, 0.f, 0.f, 0.f}, acc1 = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int st = 0; st < 8; ++st) {
    const int c = wave * 128 + st * 16 + 4 * q;
    const float4 a = *reinterpret_cast<const float4*>(xt + i * HID_STRIDE + c);
    const float4 b = *reinterpret_cast<const float4*>(wt + i * HID_STRIDE + c);
    acc0 = __builtin_amdgcn_mfma_f32_16x16x4f32(a.x, b.x, acc0, 0, 0, 0);
    acc1 = __builtin_amdgcn_mfma_f32_16x16x4f32(a.y, b.y, acc1, 0, 0, 0);
    acc0 = __builtin_amdgcn_mfma_f32_16x16x4f32(a.z, b.z, acc0, 0, 0, 0);
    acc1 = __builtin_amdgcn_mfma_f32_16x16x4f32(a.w, b.w, acc1, 0, 0, 0);
  }
  const f32x4_t acc = acc0 + acc1;
  if (wave > 0) {
#pragma unroll
    for (int r = 0; r < 4; ++r) red[wave - 1][r][lane] = acc[r];
  }
  __syncthreads();
  if (wave == 0) {
    const int j = h0 + i;                                  // result column i, rows 4q + r
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const float v = ((acc[r] + red[0][r][lane]) + red[1][r][lane]) + red[2][r][lane];
      const int sm = s0 + 4 * q + r;
      if (sm < S && j < Hd) part[(size_t(kz) * S + sm) * Hd + j] = v;
    }
  }
}

// Features of sample s for the last layer: the pooled input itself, or relu(b1 + the hidden layer's
// k-slices added in order).
static __device__ __forceinline__ float4 feature4(const float* __restrict__ feat, int nslices, size_t slice_stride,
                                                  const float* __restrict__ b1, size_t off, int d) {
  float4 p = *reinterpret_cast<const float4*>(feat + off);
  if (nslices > 0) {
#pragma unroll 8
    for (int z = 1; z < nslices; ++z) {
      const float4 t = *reinterpret_cast<const float4*>(feat + z * slice_stride + off);
      p.x += t.x; p.y += t.y; p.z += t.z; p.w += t.w;
    }
    if (b1) { const float4 t = *reinterpret_cast<const float4*>(b1 + d); p.x += t.x; p.y += t.y; p.z += t.z; p.w += t.w; }
    p.x = fmaxf(p.x, 0.f); p.y = fmaxf(p.y, 0.f); p.z = fmaxf(p.z, 0.f); p.w = fmaxf(p.w, 0.f);
  }
  return p;
}

// One sample per wave (any batch size): logits[s][k] = b2[k] + <w2[k,:], f_s> and the first index of
// the maximum.  KP = number of experts rounded up to 4, 8 or 16: all loops have fixed bounds, and
// the KP cross-lane sums advance together so that their shuffles overlap.
template <int KP>
__global__ __launch_bounds__(256) void k_router_logits_argmax(const float* __restrict__ feat, int nslices, size_t slice_stride,
                                                               const float* __restrict__ b1, const float* __restrict__ w2,
                                                               const float* __restrict__ b2, int S, int Dk, int K,
                                                               int32_t* __restrict__ expert_idx, float* __restrict__ logits) {
  const int lane = threadIdx.x & 63;
  const int s = blockIdx.x * 4 + (threadIdx.x >> 6);
  if (s >= S) return;
  // every feature is formed once (its slices are added here) and meets all K weight rows
  float acc[KP];
#pragma unroll
  for (int k = 0; k < KP; ++k) acc[k] = 0.f;
  for (int d = lane * 4; d < Dk; d += 256) {
    const float4 p = feature4(feat, nslices, slice_stride, b1, size_t(s) * Dk + d, d);
#pragma unroll
    for (int k = 0; k < KP; ++k) {
      const float4 w = *reinterpret_cast<const float4*>(w2 + size_t(k < K ? k : 0) * Dk + d);     // rows past K: row 0, unused
      acc[k] += w.x * p.x + w.y * p.y + w.z * p.z + w.w * p.w;
    }
  }
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) {
#pragma unroll
    for (int k = 0; k < KP; ++k) acc[k] += __shfl_xor(acc[k], off, 64);
  }
  float best = 0.f;
  int best_k = 0;
#pragma unroll
  for (int k = 0; k < KP; ++k) {
    if (k < K) {
      const float z = acc[k] + (b2 ? b2[k] : 0.f);
      if (logits && lane == 0) logits[size_t(s) * K + k] = z;
      if (k == 0 || z > best) { best = z; best_k = k; }   // strict >: ties keep the lowest index
    }
  }
  if (lane == 0) expert_idx[s] = best_k;
}

static void launch_logits_argmax(const float* feat, int nslices, size_t stride, const moqe_router& r, int S, int Dk,
                                 int32_t* idx, float* logits, hipStream_t st) {
  const dim3 grid((S + 3) / 4), block(256);
  const int K = r.n_experts;
  if (K <= 4) hipLaunchKernelGGL(k_router_logits_argmax<4>, grid, block, 0, st, feat, nslices, stride, r.b1, r.w2, r.b2, S, Dk, K, idx, logits);
  else if (K <= 8) hipLaunchKernelGGL(k_router_logits_argmax<8>, grid, block, 0, st, feat, nslices, stride, r.b1, r.w2, r.b2, S, Dk, K, idx, logits);
  else hipLaunchKernelGGL(k_router_logits_argmax<16>, grid, block, 0, st, feat, nslices, stride, r.b1, r.w2, r.b2, S, Dk, K, idx, logits);
}

// Logits, top-1 and the stable bucketing in ONE work-group (small batches: saves launches).
// A single work-group cannot hide latency behind other waves, so the kernel avoids chains of
// dependent accesses: all loads of a hidden-layer slice are issued together, features and last-
// layer weights sit in LDS, every (sample, expert) dot product belongs to one thread (independent
// 16-byte LDS reads, no cross-lane reductions), the chosen experts stay in LDS for the bucketing,
// and results are only stored.  NT threads share the staging (a division per group of features) and the dot products; the first four
// waves do the bucketing.  Above TAIL_SMALL_FEAT features sixteen waves: 256 samples of 64, K = 4, 9.5 us with four waves, 6.3; 40 of 384,
// K = 8, 11.0 and 8.8; 32 of 256, K = 3, 5.8 and 6.0.
// Needs S * K <= TAIL_MAX_PAIRS, S * (Dk + 4) <= TAIL_FEAT_FLOATS, S * Dk <= TAIL_MAX_FEAT and
// K * (Dk + 4) <= TAIL_MAX_W2.
constexpr int TAIL_SMALL_FEAT = 8192, TAIL_MAX_FEAT = 16384;
constexpr int TAIL_FEAT_FLOATS = 16384 + 4096;
constexpr int TAIL_MAX_W2 = 4096 + 64;     // last-layer weights (rows padded by four floats)
constexpr int TAIL_MAX_PAIRS = 2048;       // (sample, expert) pairs
constexpr int TAIL_MAX_S = 1024;
constexpr int TAIL_LDS_BYTES = (TAIL_FEAT_FLOATS + TAIL_MAX_W2 + TAIL_MAX_PAIRS + TAIL_MAX_S) * 4;

template <int NT>
__global__ __launch_bounds__(NT) void k_router_tail(const float* __restrict__ feat, int nslices, size_t slice_stride,
                                                      const float* __restrict__ b1, const float* __restrict__ w2,
                                                      const float* __restrict__ b2, int S, int Dk, int K,
                                                      int32_t* __restrict__ expert_idx, float* __restrict__ logits,
                                                      int32_t* __restrict__ counts, int32_t* __restrict__ offsets,
                                                      int32_t* __restrict__ perm, int32_t* __restrict__ inv_perm) {
  constexpr int TAIL_EPT = TAIL_MAX_FEAT / (4 * NT);      // float4 feature elements per thread, at most
  extern __shared__ __align__(16) float tail_lds[];
  float* fl = tail_lds;                                   // [S][Dk + 4]
  float* wl = tail_lds + TAIL_FEAT_FLOATS;                // [K][Dk + 4]
  float* zl = wl + TAIL_MAX_W2;                           // [S][K] logits
  int32_t* idx_l = reinterpret_cast<int32_t*>(zl + TAIL_MAX_PAIRS);
  const int tid = threadIdx.x;
  const int FS = Dk + 4;
  const int nel = S * Dk;
  for (int i = tid * 4; i < K * Dk; i += 4 * NT) {
    const int k = i / Dk, d = i - k * Dk;
    *reinterpret_cast<float4*>(wl + k * FS + d) = *reinterpret_cast<const float4*>(w2 + i);
  }
  // features: element e of this thread is the float4 at flat index 4 * (tid + NT e)
  float4 acc[TAIL_EPT];
#pragma unroll
  for (int e = 0; e < TAIL_EPT; ++e) {
    const int i = (tid + NT * e) * 4;
    acc[e] = make_float4(0.f, 0.f, 0.f, 0.f);
    if (i < nel) acc[e] = *reinterpret_cast<const float4*>(feat + i);
  }
  for (int z = 1; z < nslices; ++z) {                     // slices of the hidden layer, added in order
    const float* fz = feat + z * slice_stride;
#pragma unroll
    for (int e = 0; e < TAIL_EPT; ++e) {
      const int i = (tid + NT * e) * 4;
      if (i < nel) {
        const float4 t = *reinterpret_cast<const float4*>(fz + i);
        acc[e].x += t.x; acc[e].y += t.y; acc[e].z += t.z; acc[e].w += t.w;
      }
    }
  }
#pragma unroll
  for (int e = 0; e < TAIL_EPT; ++e) {
    const int i = (tid + NT * e) * 4;
    if (i < nel) {
      const int sm = i / Dk, d = i - sm * Dk;
      float4 p = acc[e];
      if (nslices > 0) {                                  // hidden layer: bias and ReLU
        if (b1) { const float4 t = *reinterpret_cast<const float4*>(b1 + d); p.x += t.x; p.y += t.y; p.z += t.z; p.w += t.w; }
        p.x = fmaxf(p.x, 0.f); p.y = fmaxf(p.y, 0.f); p.z = fmaxf(p.z, 0.f); p.w = fmaxf(p.w, 0.f);
      }
      *reinterpret_cast<float4*>(fl + sm * FS + d) = p;
    }
  }
  __syncthreads();
  for (int pr = tid; pr < S * K; pr += NT) {
    const int sm = pr / K, k = pr - sm * K;
    const float4* f = reinterpret_cast<const float4*>(fl + sm * FS);
    const float4* w = reinterpret_cast<const float4*>(wl + k * FS);
    float a0 = 0.f, a1 = 0.f, a2 = 0.f, a3 = 0.f;
    for (int d = 0; d < Dk / 4; ++d) {
      const float4 fv = f[d], wv = w[d];
      a0 += wv.x * fv.x; a1 += wv.y * fv.y; a2 += wv.z * fv.z; a3 += wv.w * fv.w;
    }
    const float z = ((a0 + a1) + (a2 + a3)) + (b2 ? b2[k] : 0.f);
    zl[pr] = z;
    if (logits) logits[pr] = z;
  }
  __syncthreads();
  for (int sm = tid; sm < S; sm += NT) {
    float best = zl[sm * K];
    int best_k = 0;
    for (int k = 1; k < K; ++k) {
      const float z = zl[sm * K + k];
      if (z > best) { best = z; best_k = k; }               // strict >: ties keep the lowest index
    }
    idx_l[sm] = best_k;
    expert_idx[sm] = best_k;
  }
  __syncthreads();
  if (tid >= 256) return;                                  // whole waves: the barriers from here on are met by those that are left
  bucket_body(idx_l, S, K, counts, offsets, perm, inv_perm);
}

// The whole router of a small batch without a hidden layer in ONE work-group: pooling, logits, top-1 and (offsets given) the stable bucketing.  A thread
// takes eight columns of a sample, or a share of its rows where there are fewer of those than threads (the shares are added in order); a (sample, expert)
// dot product belongs to up to sixteen neighbouring lanes.  Everything is asked for at once, so that the kernel is little more than a launch, a trip
// to memory and the barriers of the bucketing (linear block of 32 x 16 rows of 256, K = 3: 17.4 -> 14.2 us; one row of 1024 13.0 -> 10.0).  What bounds it is one
// CU issuing for sixteen waves: a thousand instructions of each are some 6 us, so there are no integer divisions and no instance for every T.
constexpr int ONE_NT = 1024;
constexpr int ONE_MAX_ELEMS = 1 << 18, ONE_MAX_NARROW = 3 << 16;     // rows x columns
constexpr int ONE_MAX_MACS = 49152;        // of the dot products
// i / d by the reciprocal of d, for 0 <= i < 2^17: (i + 1/2) / d is at least 1 / (2 d) from a whole number, the two roundings move it by less.  (An integer
// division is some forty instructions, and one CU issues them for sixteen waves.)
static __device__ __forceinline__ int quotient(int i, float inv_d) { return int((float(i) + 0.5f) * inv_d); }
constexpr int ONE_LDS_BYTES = TAIL_LDS_BYTES + ONE_NT * 32;
__global__ __launch_bounds__(ONE_NT) void k_route_one(const uint16_t* __restrict__ x, const float* __restrict__ w2, const float* __restrict__ b2, int S, int T,
                                                       int D, int K, int32_t* __restrict__ expert_idx, float* __restrict__ logits,
                                                       int32_t* __restrict__ counts, int32_t* __restrict__ offsets, int32_t* __restrict__ perm,
                                                       int32_t* __restrict__ inv_perm) {
  extern __shared__ __align__(16) float tail_lds[];
  float* fl = tail_lds;                                   // [S][D + 4]
  float* wl = tail_lds + TAIL_FEAT_FLOATS;                // [K][D + 4]
  float* zl = wl + TAIL_MAX_W2;                           // [S][K] logits
  int32_t* idx_l = reinterpret_cast<int32_t*>(zl + TAIL_MAX_PAIRS);
  float* red = reinterpret_cast<float*>(idx_l + TAIL_MAX_S);          // [shares][S][D]
  const int tid = threadIdx.x, FS = D + 4, c8 = D >> 3, tasks = S * c8;
  int shares = 1;
  while (shares * 2 * tasks <= ONE_NT && shares < T) shares <<= 1;
  const float per_task = __frcp_rn(float(tasks)), per_c8 = __frcp_rn(float(c8)), per_d = __frcp_rn(float(D)), rows = float(T);
  const int share = shares > 1 ? quotient(tid, per_task) : 0, first = tid - share * tasks;
  for (int i = tid * 4; i < K * D; i += 4 * ONE_NT) {
    const int k = quotient(i, per_d);
    *reinterpret_cast<float4*>(wl + i + 4 * k) = *reinterpret_cast<const float4*>(w2 + i);
  }
#pragma unroll 1
  for (int i = first; i < tasks && share < shares; i += ONE_NT) {     // one turn where rows are shared out
    const int sm = quotient(i, per_c8), c = (i - sm * c8) * 8;
    const uint16_t* p = x + (size_t(sm) * T + share) * D + c;
    const size_t step = size_t(shares) * D;
    float acc[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    auto add = [&](const uint4& v) {
      const uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        acc[2 * j] += __uint_as_float(w[j] << 16);
        acc[2 * j + 1] += __uint_as_float(w[j] & 0xffff0000u);
      }
    };
    int t = share;
#pragma unroll 1
    for (; t + 7 * shares < T; t += 8 * shares) {         // eight rows in flight
      uint4 v[8];
#pragma unroll
      for (int u = 0; u < 8; ++u, p += step) v[u] = *reinterpret_cast<const uint4*>(p);
#pragma unroll
      for (int u = 0; u < 8; ++u) add(v[u]);
    }
#pragma unroll 1
    for (; t < T; t += 2 * shares) {                      // the rest, two at a time
      const bool two = t + shares < T;
      const uint4 a = *reinterpret_cast<const uint4*>(p), b = *reinterpret_cast<const uint4*>(two ? p + step : p);
      p += 2 * step;
      add(a);
      if (two) add(b);
    }
    float* f = shares > 1 ? red + (share * tasks + i) * 8 : fl + sm * FS + c;
    if (shares == 1 && T > 1) {
#pragma unroll
      for (int j = 0; j < 8; ++j) acc[j] = __fdiv_rn(acc[j], rows);
    }
    *reinterpret_cast<float4*>(f) = make_float4(acc[0], acc[1], acc[2], acc[3]);
    *reinterpret_cast<float4*>(f + 4) = make_float4(acc[4], acc[5], acc[6], acc[7]);
  }
  __syncthreads();
  if (shares > 1) {                                       // the shares in order, and the mean
    const int n = S * D;
#pragma unroll 1
    for (int i = tid; i < n; i += ONE_NT) {
      float v = red[i];
      for (int r = 1; r < shares; ++r) v += red[r * n + i];
      fl[i + 4 * quotient(i, per_d)] = __fdiv_rn(v, rows);
    }
    __syncthreads();
  }
  int lanes_log2 = 0;                                     // lanes of a dot product
  while (lanes_log2 < 4 && (2 << lanes_log2) * S * K <= ONE_NT) ++lanes_log2;
  const int lanes = 1 << lanes_log2;
  const float per_k = __frcp_rn(float(K));
  for (int i = tid; i < S * K * lanes; i += ONE_NT) {     // whole groups of lanes together: ONE_NT is a multiple of sixteen
    const int l = i & (lanes - 1), pr = i >> lanes_log2, sm = quotient(pr, per_k), k = pr - sm * K;
    const float4* f = reinterpret_cast<const float4*>(fl + sm * FS);
    const float4* w = reinterpret_cast<const float4*>(wl + k * FS);
    float a0 = 0.f, a1 = 0.f, a2 = 0.f, a3 = 0.f;
#pragma unroll 4
    for (int d = l; d < D / 4; d += lanes) {
      const float4 fv = f[d], wv = w[d];
      a0 += wv.x * fv.x; a1 += wv.y * fv.y; a2 += wv.z * fv.z; a3 += wv.w * fv.w;
    }
    float z = (a0 + a1) + (a2 + a3);
    for (int off = lanes >> 1; off >= 1; off >>= 1) z += __shfl_xor(z, off, 64);
    if (l == 0) {
      z += b2 ? b2[k] : 0.f;
      zl[pr] = z;
      if (logits) logits[pr] = z;
    }
  }
  __syncthreads();
  for (int sm = tid; sm < S; sm += ONE_NT) {
    float best = zl[sm * K];
    int best_k = 0;
    for (int k = 1; k < K; ++k) {
      const float z = zl[sm * K + k];
      if (z > best) { best = z; best_k = k; }               // strict >: ties keep the lowest index
    }
    idx_l[sm] = best_k;
    expert_idx[sm] = best_k;
  }
  if (!offsets) return;                                    // uniform
  __syncthreads();
  if (tid >= 256) return;                                  // whole waves: the barriers from here on are met by those that are left
  bucket_body(idx_l, S, K, counts, offsets, perm, inv_perm);
}

// Samples of different lengths: pooled[s][d] = mean over the rows cu_rows[s] .. cu_rows[s+1] of x[., d].
// A work-group takes 8 CT columns of one sample: CT column-threads of 8 columns x 256 / CT row-threads, eight row loads in flight each (rows
// past the sample's end are clamped, loaded and taken as zeros), the row-threads' sums added in order.  A sample of at most eight rows
// is left to the first row-thread, which has them all in flight and meets no barrier.  Bound by reading x once (40 samples of up to 900
// rows of 4096: 346 us with a thread per 8 columns that walks a whole sample row by row, 13 us with CT = 16).
template <int CT>
__global__ __launch_bounds__(256) void k_pool_ragged(const uint16_t* __restrict__ x, const int32_t* __restrict__ cu_rows,
                                                      float* __restrict__ pooled, int D) {
  constexpr int TR = 256 / CT;
  __shared__ __align__(16) float red[TR][CT * 8];
  const int s = blockIdx.y;
  const int ct = threadIdx.x % CT, tr = threadIdx.x / CT;
  const int col = (blockIdx.x * CT + ct) * 8;
  const int r0 = cu_rows[s], r1 = cu_rows[s + 1], rows = r1 - r0;
  const float inv = rows > 0 ? 1.0f / float(rows) : 0.f;     // a sample without rows has all-zero features
  const uint16_t* base = x + col;
  float acc[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  auto add = [&](const uint4& v) {
    const uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      acc[2 * j] += bf16_bits_to_float(w[j] & 0xffffu);
      acc[2 * j + 1] += bf16_bits_to_float(w[j] >> 16);
    }
  };
  if (rows <= 8) {                                           // uniform over the work-group
    if (tr > 0 || col >= D) return;
    uint4 v4[8];
#pragma unroll
    for (int u = 0; u < 8; ++u)
      if (u < rows) v4[u] = *reinterpret_cast<const uint4*>(base + size_t(r0 + u) * D);
#pragma unroll
    for (int u = 0; u < 8; ++u)
      if (u < rows) add(v4[u]);
    float4* dst = reinterpret_cast<float4*>(pooled + size_t(s) * D + col);
    dst[0] = make_float4(acc[0] * inv, acc[1] * inv, acc[2] * inv, acc[3] * inv);
    dst[1] = make_float4(acc[4] * inv, acc[5] * inv, acc[6] * inv, acc[7] * inv);
    return;
  }
  if (col < D) {
    int r = r0 + tr;
    uint4 v4[8];
    for (; r + 7 * TR < r1; r += 8 * TR) {
#pragma unroll
      for (int u = 0; u < 8; ++u) v4[u] = *reinterpret_cast<const uint4*>(base + size_t(r + u * TR) * D);
#pragma unroll
      for (int u = 0; u < 8; ++u) add(v4[u]);
    }
    if (r < r1) {                                            // the rest: selected, not branched over, or loads would sink behind the branches
#pragma unroll
      for (int u = 0; u < 8; ++u) v4[u] = *reinterpret_cast<const uint4*>(base + size_t(min(r + u * TR, r1 - 1)) * D);
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        const uint32_t keep = r + u * TR < r1 ? 0xffffffffu : 0u;
        add(make_uint4(v4[u].x & keep, v4[u].y & keep, v4[u].z & keep, v4[u].w & keep));
      }
    }
  }
#pragma unroll
  for (int i = 0; i < 8; ++i) red[tr][ct * 8 + i] = acc[i];
  __syncthreads();
  for (int i = threadIdx.x; i < CT * 8; i += 256) {
    const int c = blockIdx.x * (CT * 8) + i;
    if (c >= D) continue;
    float v = red[0][i];
#pragma unroll
    for (int t = 1; t < TR; ++t) v += red[t][i];
    pooled[size_t(s) * D + c] = v * inv;
  }
}

// Chunks of a sample's tokens (C) and column-threads per work-group (CT).  A batch that fills the chip with one
// work-group per sample and column block, and whose samples are short, is pooled in one chunk - and then in one launch.
static void pool_shape(int S, int T, int D, int* C, int* CT) {
  int cols8 = D / 8;
  int ct = 1;
  while (ct < cols8 && ct < 256) ct <<= 1;
  int c = T / 64;
  if (c < 1) c = 1;
  if (c > 16) c = 16;
  if (T <= 256 && long(S) * ((cols8 + ct - 1) / ct) >= 256) c = 1;
  // Two work-groups to a CU at least: narrower column blocks, more rows at a time (the router alone: 128 x 256 rows of 3584 53.6 -> 48.5 us, 40 x 300 of 2048
  // 24.8 -> 21.7, 8 x 700 of 4096 26.3 -> 23.9; with four to a CU 49.4, 21.4 and 23.3, but 16 x 512 of 4096 28.6, with two 26.4 for 27.5).  Only while a
  // thread keeps its eight rows in flight: few rows are better walked by one row of threads than summed over many (2 x 3 rows of 1664, a linear block 12.5 us
  // for 14.2).
  while (ct > 16 && (T + c - 1) / c * ct >= 4096 && long(S) * c * ((cols8 + ct - 1) / ct) < 512) ct >>= 1;
  *CT = ct;
  *C = c;
}

static int hidden_slices(int D) { return (D + HID_KC - 1) / HID_KC; }

size_t route_ws_bytes(int S, int T, const moqe_router& r) {
  int C, CT;
  pool_shape(S, T, r.d, &C, &CT);
  size_t b = align256(size_t(S) * C * r.d * 4);                   // partial sums of the pooling
  b += align256(size_t(S) * r.d * 4);                             // pooled features
  b += align256(size_t(hidden_slices(r.d)) * S * (r.h > 0 ? r.h : 1) * 4);   // hidden layer, one slab per k-slice
  return b;
}

// Pooling and hidden layer; returns the feature description for the logits stage.
struct RouteFeat { const float* feat; int nslices; size_t stride; int Dk; };

static int32_t route_front(const void* x, const int32_t* cu_rows, int S, int T, const moqe_router& r, void* ws, hipStream_t st,
                           RouteFeat* rf) {
  int C, CT;
  pool_shape(S, T, r.d, &C, &CT);
  const int D = r.d;
  uint8_t* p = static_cast<uint8_t*>(ws);
  float* partial = reinterpret_cast<float*>(p);
  p += align256(size_t(S) * C * D * 4);
  float* pooled = reinterpret_cast<float*>(p);
  p += align256(size_t(S) * D * 4);
  float* hidden = reinterpret_cast<float*>(p);
  const bool direct = (!cu_rows && T == 1 && r.h > 0);      // the hidden layer reads the bf16 rows themselves
  if (cu_rows) {
    ProfileScope ps(MOQE_PK_ROUTE, st);
    const uint16_t* xr = static_cast<const uint16_t*>(x);
    auto go = [&](auto kernel, int ct) { hipLaunchKernelGGL(kernel, dim3((D / 8 + ct - 1) / ct, S), dim3(256), 0, st, xr, cu_rows, pooled, D); };
    // Few samples: narrow column blocks, many rows at a time, so that a long sample is spread over the chip (40 samples of up to 900 rows of
    // 4096: 21 us with 16 column-threads, 29 with 32).  Many samples fill the chip by themselves, and where they are short what is
    // left is the dispatch of work-groups: 5000 samples of one or two rows of 4096 take 82 us with 16 and 51 with 64 (a thread per 8
    // columns that walks its sample: 50), 1000 of 1 to 4 26 and 20, of 8192 columns 42 and 31, 28 with 128; 256 of 1 to 4 rows of 1024
    // 9.6 and, with 32, 9.1.  On samples of 60 to 300 rows the widths differ by 2 to 5 %.
    const long vecs = S >= 200 ? long(S) * (D / 8) : 0;
    if (vecs >= 1000000) go(k_pool_ragged<128>, 128);
    else if (vecs >= 60000) go(k_pool_ragged<64>, 64);
    else if (vecs >= 32000) go(k_pool_ragged<32>, 32);
    else go(k_pool_ragged<16>, 16);
  } else if (!direct) {
    {
      ProfileScope ps(MOQE_PK_ROUTE, st);
      dim3 grid((D / 8 + CT - 1) / CT, C, S);
      hipLaunchKernelGGL(k_pool_partial, grid, dim3(256), 0, st, static_cast<const uint16_t*>(x), C == 1 ? pooled : partial, T, D, C,
                         CT, C == 1 ? 1 : 0);
    }
    if (C > 1) {
      ProfileScope ps(MOQE_PK_ROUTE, st);
      size_t nel = size_t(S) * D;
      hipLaunchKernelGGL(k_pool_finish, dim3(unsigned((nel + 255) / 256)), dim3(256), 0, st, partial, pooled, S, T, D, C);
    }
  }
  if (r.h > 0) {
    const int KS = hidden_slices(D);
    ProfileScope ps(MOQE_PK_ROUTE, st);
    dim3 grid((r.h + 15) / 16, (S + 15) / 16, KS);
    if (direct) hipLaunchKernelGGL(k_router_hidden<true>, grid, dim3(256), 0, st, x, r.w1, hidden, S, D, r.h);
    else hipLaunchKernelGGL(k_router_hidden<false>, grid, dim3(256), 0, st, static_cast<const void*>(pooled), r.w1, hidden, S, D, r.h);
    *rf = RouteFeat{hidden, KS, size_t(S) * r.h, r.h};
  } else {
    *rf = RouteFeat{pooled, 0, 0, D};
  }
  return check_launch("route");
}

// One work-group for the whole router: no hidden layer, and little enough that a CU's loads and LDS reads do not outweigh the two launches saved (linear
// blocks, us before / after): rows x columns up to 2^18 (16 x 16 of 1024, K = 3 35.2 / 27.0; 11 x 22 of 1024, K = 4 39.4 / 29.9), narrow samples, whose
// former launches are short, up to 3 * 2^16 (81 x 16 of 128 18.2 / 16.4; with more 47 x 21 of 256, K = 4 20.5 / 21.3, 128 x 15 of 128 18.9 / 19.5), and
// samples x experts x columns up to 49152 (46 x 10 of 256, K = 3 20.7 / 17.2; 60 x 2 of 256, K = 4 17.4 / 18.7; 64 x 16 of 256, K = 8 23.0 / 24.3).
static bool route_one_fits(int S, int T, const moqe_router& r) {
  return r.h == 0 && r.d % 8 == 0 && S <= TAIL_MAX_S && S * r.n_experts <= TAIL_MAX_PAIRS && size_t(S) * (r.d + 4) <= size_t(TAIL_FEAT_FLOATS) &&
         r.n_experts * (r.d + 4) <= TAIL_MAX_W2 && size_t(S) * T * r.d <= size_t(r.d <= 256 ? ONE_MAX_NARROW : ONE_MAX_ELEMS) && size_t(S) * r.n_experts * r.d <= size_t(ONE_MAX_MACS);
}
static int32_t launch_route_one(const void* x, int S, int T, const moqe_router& r, int32_t* idx, float* logits, int32_t* counts, int32_t* offsets, int32_t* perm,
                                int32_t* inv_perm, hipStream_t st) {
  const int32_t rc = ensure_dynamic_lds(LDSK_ROUTE_ONE, reinterpret_cast<const void*>(&k_route_one), ONE_LDS_BYTES, "route");
  if (rc) return rc;
  ProfileScope ps(MOQE_PK_ROUTE, st);
  hipLaunchKernelGGL(k_route_one, dim3(1), dim3(ONE_NT), ONE_LDS_BYTES, st, static_cast<const uint16_t*>(x), r.w2, r.b2, S, T, r.d, r.n_experts, idx, logits, counts,
                     offsets, perm, inv_perm);
  return check_launch("route");
}

int32_t launch_route(const void* x, int S, int T, const moqe_router& r, int32_t* idx, float* logits,
                     void* ws, hipStream_t st) {
  if (route_one_fits(S, T, r)) return launch_route_one(x, S, T, r, idx, logits, nullptr, nullptr, nullptr, nullptr, st);
  RouteFeat rf;
  int32_t rc = route_front(x, nullptr, S, T, r, ws, st, &rf);
  if (rc) return rc;
  ProfileScope ps(MOQE_PK_ROUTE, st);
  launch_logits_argmax(rf.feat, rf.nslices, rf.stride, r, S, rf.Dk, idx, logits, st);
  return check_launch("route");
}

// The router's MLP on feature vectors that are already there (feat: fp32 [S, r.d]); workspace route_ws_bytes(S, 1, r).
int32_t launch_route_features(const float* feat, int S, const moqe_router& r, int32_t* idx, float* logits, void* ws, hipStream_t st) {
  RouteFeat rf{feat, 0, 0, r.d};
  if (r.h > 0) {
    int C, CT;
    pool_shape(S, 1, r.d, &C, &CT);
    float* hidden = reinterpret_cast<float*>(static_cast<uint8_t*>(ws) + align256(size_t(S) * C * r.d * 4) + align256(size_t(S) * r.d * 4));
    const int KS = hidden_slices(r.d);
    ProfileScope ps(MOQE_PK_ROUTE, st);
    hipLaunchKernelGGL(k_router_hidden<false>, dim3((r.h + 15) / 16, (S + 15) / 16, KS), dim3(256), 0, st,
                       static_cast<const void*>(feat), r.w1, hidden, S, r.d, r.h);
    rf = RouteFeat{hidden, KS, size_t(S) * r.h, r.h};
  }
  ProfileScope ps(MOQE_PK_ROUTE, st);
  launch_logits_argmax(rf.feat, rf.nslices, rf.stride, r, S, rf.Dk, idx, logits, st);
  return check_launch("route");
}

// Samples of different lengths (cu_rows: device int32 [S + 1], first row of every sample): the
// workspace is that of route_ws_bytes(S, 2, r).
int32_t launch_route_ragged(const void* x, const int32_t* cu_rows, int S, const moqe_router& r, int32_t* idx, float* logits,
                            void* ws, hipStream_t st) {
  RouteFeat rf;
  int32_t rc = route_front(x, cu_rows, S, 2, r, ws, st, &rf);
  if (rc) return rc;
  ProfileScope ps(MOQE_PK_ROUTE, st);
  launch_logits_argmax(rf.feat, rf.nslices, rf.stride, r, S, rf.Dk, idx, logits, st);
  return check_launch("route");
}

// Router and bucketing together; small batches finish in one work-group.
int32_t launch_route_bucket(const void* x, int S, int T, const moqe_router& r, int32_t* idx, float* logits,
                            int32_t* counts, int32_t* offsets, int32_t* perm, int32_t* inv_perm, void* ws, hipStream_t st) {
  const int Dk = r.h > 0 ? r.h : r.d;
  if (route_one_fits(S, T, r)) return launch_route_one(x, S, T, r, idx, logits, counts, offsets, perm, inv_perm, st);
  if (S > TAIL_MAX_S || S * r.n_experts > TAIL_MAX_PAIRS || size_t(S) * (Dk + 4) > size_t(TAIL_FEAT_FLOATS) ||
      size_t(S) * Dk > size_t(TAIL_MAX_FEAT) || r.n_experts * (Dk + 4) > TAIL_MAX_W2) {
    int32_t rc = launch_route(x, S, T, r, idx, logits, ws, st);
    if (rc) return rc;
    return launch_bucket(idx, S, r.n_experts, counts, offsets, perm, inv_perm, st);
  }
  RouteFeat rf;
  int32_t rc = route_front(x, nullptr, S, T, r, ws, st, &rf);
  if (rc) return rc;
  if (rf.nslices > 1) {
    // the slices of the hidden layer are best added by many work-groups: separate logits and bucket kernels
    {
      ProfileScope ps(MOQE_PK_ROUTE, st);
      launch_logits_argmax(rf.feat, rf.nslices, rf.stride, r, S, rf.Dk, idx, logits, st);
    }
    return launch_bucket(idx, S, r.n_experts, counts, offsets, perm, inv_perm, st);
  }
  const bool small = S * rf.Dk <= TAIL_SMALL_FEAT;
  const auto kernel = small ? k_router_tail<256> : k_router_tail<1024>;
  rc = ensure_dynamic_lds(LDSK_ROUTER_TAIL + (small ? 0 : 1), reinterpret_cast<const void*>(kernel), TAIL_LDS_BYTES, "route");
  if (rc) return rc;
  ProfileScope ps(MOQE_PK_BUCKET, st);
  hipLaunchKernelGGL(kernel, dim3(1), dim3(small ? 256 : 1024), TAIL_LDS_BYTES, st, rf.feat, rf.nslices, rf.stride, r.b1, r.w2,
                     r.b2, S, rf.Dk, r.n_experts, idx, logits, counts, offsets, perm, inv_perm);
  return check_launch("route+bucket");
}

}  // namespace moqe
