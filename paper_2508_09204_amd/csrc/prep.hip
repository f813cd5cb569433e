// Weight preparation and activation preparation kernels:
//   round-to-nearest quantizers (canonical layout), canonical <-> packed layout,
//   per-row dynamic int8 activation quantization (W8A8 expert).
// The quantizers use fp32 IEEE operations with explicit rounding intrinsics so that no
// multiply-add contraction changes a code.
#include "moqe_internal.h"

#include <algorithm>

namespace moqe {

static __device__ __forceinline__ float wave_max(float v) {
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) v = fmaxf(v, __shfl_xor(v, off, 64));
  return v;
}

// Block-wide max of non-negative values, every thread gets the result.
static __device__ __forceinline__ float block_max_256(float v, float* sh) {
  v = wave_max(v);
  if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = v;
  __syncthreads();
  float r = fmaxf(fmaxf(sh[0], sh[1]), fmaxf(sh[2], sh[3]));
  __syncthreads();
  return r;
}

// Pointers of the canonical layout carry no alignment promise: these types are loaded and stored with one (unaligned) access.
typedef float f32x4_any __attribute__((ext_vector_type(4), aligned(4)));
typedef uint32_t u32_any __attribute__((aligned(1)));
typedef uint32_t u32x2_any __attribute__((ext_vector_type(2), aligned(1)));
typedef uint32_t u32x4_any __attribute__((ext_vector_type(4), aligned(1)));

// ---- symmetric per-output-channel: one work-group per row ---------------------------------
// Bound by reading w once: 16-byte loads, and a row of up to 12288 columns stays in registers between the maximum and the codes
// (mean over the 8-bit matrices of a 4096 / 11008 and a 3584 / 18944 block: 35 us; with 4-byte loads and a second read 72 us on the first).
constexpr int QS_VEC = 12;               // vectors of four per thread
__global__ __launch_bounds__(256) void k_quant_sym(const float* __restrict__ w, int n, int k, int bits,
                                                    int8_t* __restrict__ q, float* __restrict__ scale) {
  __shared__ float sh[4];
  const int row = blockIdx.x;
  const float* wr = w + size_t(row) * k;
  f32x4_any v[QS_VEC];
  float a = 0.f;
#pragma unroll
  for (int i = 0; i < QS_VEC; ++i) {
    const int c = (i * 256 + threadIdx.x) * 4;               // k is a multiple of 128
    v[i] = c < k ? *reinterpret_cast<const f32x4_any*>(wr + c) : f32x4_any{0.f, 0.f, 0.f, 0.f};
  }
  auto top = [&](const f32x4_any& x) { a = fmaxf(a, fmaxf(fmaxf(fabsf(x.x), fabsf(x.y)), fmaxf(fabsf(x.z), fabsf(x.w)))); };
#pragma unroll
  for (int i = 0; i < QS_VEC; ++i) top(v[i]);
  for (int c = (QS_VEC * 256 + threadIdx.x) * 4; c < k; c += 1024) top(*reinterpret_cast<const f32x4_any*>(wr + c));
  a = block_max_256(a, sh);
  const float qmax = float((1 << (bits - 1)) - 1);
  const float s = (a == 0.f) ? 1.0f : __fdiv_rn(a, qmax);
  if (threadIdx.x == 0) scale[row] = s;
  int8_t* qr = q + size_t(row) * k;
  auto code = [&](float x) {
    const float t = fminf(fmaxf(rintf(__fdiv_rn(x, s)), -qmax), qmax);
    return uint32_t(uint8_t(int8_t(int(t))));
  };
  auto put = [&](int c, const f32x4_any& x) {
    *reinterpret_cast<u32_any*>(qr + c) = code(x.x) | code(x.y) << 8 | code(x.z) << 16 | code(x.w) << 24;
  };
#pragma unroll
  for (int i = 0; i < QS_VEC; ++i) {
    const int c = (i * 256 + threadIdx.x) * 4;
    if (c < k) put(c, v[i]);
  }
  for (int c = (QS_VEC * 256 + threadIdx.x) * 4; c < k; c += 1024) put(c, *reinterpret_cast<const f32x4_any*>(wr + c));
}

// ---- asymmetric group-wise: GROUP / 4 lanes per group, four values each ------------------------
// Groups are consecutive in memory (k is a multiple of the group), so the kernel walks them as one list; a wave has QA_VEC loads of
// 1 KiB in flight (11008 x 4096, groups of 128: 43 us; with a wave per group and 4-byte loads 119 us).
constexpr int QA_VEC = 4;
template <int GROUP>
__global__ __launch_bounds__(256) void k_quant_asym(const float* __restrict__ w, size_t groups, int bits, float clip,
                                                     uint8_t* __restrict__ q, float* __restrict__ scale, uint8_t* __restrict__ zero) {
  constexpr int LPG = GROUP / 4, GPW = 64 / LPG;             // lanes per group, groups per wave and load
  const int lane = threadIdx.x & 63, gl = lane % LPG;
  const size_t g0 = (size_t(blockIdx.x) * 4 + (threadIdx.x >> 6)) * (GPW * QA_VEC) + lane / LPG;
  f32x4_any v[QA_VEC];
#pragma unroll
  for (int u = 0; u < QA_VEC; ++u) {
    const size_t gid = g0 + u * GPW;
    v[u] = gid < groups ? *reinterpret_cast<const f32x4_any*>(w + gid * GROUP + gl * 4) : f32x4_any{0.f, 0.f, 0.f, 0.f};
  }
#pragma unroll
  for (int u = 0; u < QA_VEC; ++u) {
    const size_t gid = g0 + u * GPW;
    float mn = fminf(0.f, fminf(fminf(v[u].x, v[u].y), fminf(v[u].z, v[u].w)));
    float mx = fmaxf(0.f, fmaxf(fmaxf(v[u].x, v[u].y), fmaxf(v[u].z, v[u].w)));
#pragma unroll
    for (int off = LPG / 2; off >= 1; off >>= 1) {
      mn = fminf(mn, __shfl_xor(mn, off, 64));
      mx = fmaxf(mx, __shfl_xor(mx, off, 64));
    }
    const float L = float((1 << bits) - 1);
    const float lo = __fmul_rn(clip, mn), hi = __fmul_rn(clip, mx);
    const float s = (hi == lo) ? 1.0f : __fdiv_rn(__fsub_rn(hi, lo), L);
    const float z = fminf(fmaxf(rintf(__fdiv_rn(-lo, s)), 0.f), L);
    auto code = [&](float x) {
      const float t = fminf(fmaxf(__fadd_rn(rintf(__fdiv_rn(x, s)), z), 0.f), L);
      return uint32_t(uint8_t(int(t)));
    };
    if (gid < groups) {
      if (gl == 0) { scale[gid] = s; zero[gid] = uint8_t(int(z)); }
      *reinterpret_cast<u32_any*>(q + gid * GROUP + gl * 4) = code(v[u].x) | code(v[u].y) << 8 | code(v[u].z) << 16 | code(v[u].w) << 24;
    }
  }
}

int32_t launch_quantize(const float* w, float clip, const moqe_qmat& out, hipStream_t st) {
  ProfileScope ps(MOQE_PK_OTHER, st);
  if (out.symmetric) {
    hipLaunchKernelGGL(k_quant_sym, dim3(out.n), dim3(256), 0, st, w, out.n, out.k, out.bits,
                       static_cast<int8_t*>(const_cast<void*>(out.qdata)), const_cast<float*>(out.scale));
  } else {
    const size_t groups = size_t(out.n) * (out.k / out.group);
    uint8_t* q = static_cast<uint8_t*>(const_cast<void*>(out.qdata));
    float* scale = const_cast<float*>(out.scale);
    uint8_t* zero = const_cast<uint8_t*>(out.zero);
    const size_t per_wg = 4 * (256 / out.group) * QA_VEC;
    const dim3 grid(unsigned((groups + per_wg - 1) / per_wg));
    if (out.group == 128) hipLaunchKernelGGL(k_quant_asym<128>, grid, dim3(256), 0, st, w, groups, out.bits, clip, q, scale, zero);
    else hipLaunchKernelGGL(k_quant_asym<64>, grid, dim3(256), 0, st, w, groups, out.bits, clip, q, scale, zero);
  }
  return check_launch("quantize_rtn");
}

// ---- canonical -> packed -------------------------------------------------------------------
// Scales and zero-points in the blob's order, and zeros in what is left of their regions (each ends on a multiple of 256 bytes).
static __device__ __forceinline__ void pack_meta(const size_t i, const float* __restrict__ scale, const uint8_t* __restrict__ zero, int n, int k,
                                                 const PackedInfo& pi, uint8_t* __restrict__ out) {
  const size_t nscale = pi.gpt ? size_t(pi.nt) * pi.kt * 16 * pi.gpt : size_t(n);
  size_t src = i;
  if (pi.gpt) {                                              // i = (tile * 16 + row of the tile) * gpt + group of the tile
    const size_t t = i / size_t(16 * pi.gpt);
    const int r = int(i / pi.gpt) & 15, g = int(i % pi.gpt);
    src = ((t / pi.kt) * 16 + r) * size_t(k / (128 / pi.gpt)) + (t % pi.kt) * pi.gpt + g;
  }
  if (pi.scale_off + i * 4 < pi.zero_off) reinterpret_cast<float*>(out + pi.scale_off)[i] = i < nscale ? scale[src] : 0.f;
  if (pi.asym && pi.zero_off + i < pi.total) (out + pi.zero_off)[i] = i < nscale ? zero[src] : uint8_t(0);
}

// A wave per tile: lane l = kq*16 + r reads its 32 codes of row r (8 columns per matrix-core step; 16 per half for the int8-activation
// order), puts its share of the tile together in registers and stores it with 16-, 8- or 4-byte accesses that are contiguous over
// the wave.  Every byte of the blob is written, so it need not be cleared first.  (One atomic OR per code into a cleared blob, as it was:
// 2.0 ms for 11008 x 4096 in 4 bits, 13 us now.)  The work-groups behind the tiles' take the scales and zero-points: as a launch of
// their own they took 4 us after the codes, of which there is nothing to wait for (building an expert of 11008 x 4096 64.2 -> 61.1 us).
template <int FMT>
__global__ __launch_bounds__(256) void k_pack_codes(const moqe_qmat c_in, const PackedInfo pi, const unsigned code_wgs, uint8_t* __restrict__ out) {
  if (blockIdx.x >= code_wgs) {
    pack_meta(size_t(blockIdx.x - code_wgs) * 256 + threadIdx.x, c_in.scale, c_in.zero, c_in.n, c_in.k, pi, out);
    return;
  }
  const uint8_t* __restrict__ q = static_cast<const uint8_t*>(c_in.qdata);
  const int k = c_in.k, kt = pi.kt, zc = pi.zc;
  const size_t tiles = size_t(pi.nt) * pi.kt;
  const int lane = threadIdx.x & 63, r = lane & 15, kq = lane >> 4;
  const size_t t = size_t(blockIdx.x) * 4 + (threadIdx.x >> 6);
  if (t >= tiles) return;
  constexpr uint32_t TILE = FMT == FMT_I8 || FMT == FMT_I8A8 ? 2048u : FMT == FMT_N4 ? 1024u : FMT == FMT_N3 ? 768u : 1536u;
  const uint8_t* src = q + ((t / size_t(kt)) * 16 + r) * size_t(k) + (t % size_t(kt)) * 128;
  uint8_t* dst = out + t * TILE;                             // the blob is 256-byte aligned, so is every tile
  if constexpr (FMT == FMT_I8A8) {
#pragma unroll
    for (int h = 0; h < 2; ++h)
      *reinterpret_cast<uint4*>(dst + h * 1024 + lane * 16) = __builtin_bit_cast(uint4, *reinterpret_cast<const u32x4_any*>(src + 64 * h + 16 * kq));
    return;
  }
  uint32_t c[4][8];
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const u32x2_any v = *reinterpret_cast<const u32x2_any*>(src + 32 * j + 8 * kq);
#pragma unroll
    for (int i = 0; i < 8; ++i) c[j][i] = (((i < 4 ? v.x : v.y) >> (8 * (i & 3))) + uint32_t(zc)) & 0xffu;
  }
  if constexpr (FMT == FMT_I8) {
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      uint32_t d[4];
#pragma unroll
      for (int w = 0; w < 4; ++w) {
        const uint32_t* e = &c[2 * h + w / 2][(w & 1) * 4];
        d[w] = e[0] | e[1] << 8 | e[2] << 16 | e[3] << 24;
      }
      *reinterpret_cast<uint4*>(dst + h * 1024 + lane * 16) = make_uint4(d[0], d[1], d[2], d[3]);
    }
  } else {
    constexpr int PAIR = 16;                                 // odd columns live in the upper half of a dword
    uint32_t nib[4] = {0u, 0u, 0u, 0u}, two[2] = {0u, 0u}, one = 0u;
#pragma unroll
    for (int j = 0; j < 4; ++j)
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        const int up = (i & 1) * PAIR, f = i / 2;
        if constexpr (FMT == FMT_N3) {
          two[j / 2] |= (c[j][i] & 3u) << (2 * (4 * (j % 2) + f) + up);
          one |= ((c[j][i] >> 2) & 1u) << (4 * j + f + up);
        } else {
          nib[j] |= (c[j][i] & 15u) << (4 * f + up);
          if constexpr (FMT == FMT_N6) two[j / 2] |= ((c[j][i] >> 4) & 3u) << (2 * (4 * (j % 2) + f) + up);
        }
      }
    if constexpr (FMT == FMT_N3) {
      *reinterpret_cast<uint2*>(dst + lane * 8) = make_uint2(two[0], two[1]);
      *reinterpret_cast<uint32_t*>(dst + 512 + lane * 4) = one;
    } else {
      *reinterpret_cast<uint4*>(dst + lane * 16) = make_uint4(nib[0], nib[1], nib[2], nib[3]);
      if constexpr (FMT == FMT_N6) *reinterpret_cast<uint2*>(dst + 1024 + lane * 8) = make_uint2(two[0], two[1]);
    }
  }
}

int32_t launch_pack(const moqe_qmat& c, const PackedInfo& pi, uint8_t* out, hipStream_t st) {
  ProfileScope ps(MOQE_PK_OTHER, st);
  const unsigned code_wgs = unsigned((size_t(pi.nt) * pi.kt + 3) / 4);
  const size_t nmeta = std::max((pi.zero_off - pi.scale_off) / 4, pi.total - pi.zero_off);
  const dim3 grid(code_wgs + unsigned((nmeta + 255) / 256)), block(256);
  switch (pi.fmt) {
    case FMT_I8:   hipLaunchKernelGGL(k_pack_codes<FMT_I8>, grid, block, 0, st, c, pi, code_wgs, out); break;
    case FMT_I8A8: hipLaunchKernelGGL(k_pack_codes<FMT_I8A8>, grid, block, 0, st, c, pi, code_wgs, out); break;
    case FMT_N6:   hipLaunchKernelGGL(k_pack_codes<FMT_N6>, grid, block, 0, st, c, pi, code_wgs, out); break;
    case FMT_N4:   hipLaunchKernelGGL(k_pack_codes<FMT_N4>, grid, block, 0, st, c, pi, code_wgs, out); break;
    default:       hipLaunchKernelGGL(k_pack_codes<FMT_N3>, grid, block, 0, st, c, pi, code_wgs, out); break;
  }
  return check_launch("pack_qmat");
}

// ---- packed -> integer weights (code - zero) and scales in canonical shape ------------------
__global__ void k_unpack(const uint8_t* __restrict__ blob, int n, int k, PackedInfo pi, int16_t* __restrict__ out,
                         float* __restrict__ scale_out) {
  size_t i = size_t(blockIdx.x) * blockDim.x + threadIdx.x;
  if (i >= size_t(n) * k) return;
  const int row = int(i / k), col = int(i % k);
  const CodePos p = code_pos(pi, row, col);
  uint32_t code = (*reinterpret_cast<const uint32_t*>(blob + p.byte0) >> p.shift0) & ((1u << p.bits0) - 1u);
  if (p.bits1) code |= ((*reinterpret_cast<const uint32_t*>(blob + p.byte1) >> p.shift1) & ((1u << p.bits1) - 1u)) << p.bits0;
  const size_t mi = meta_index(pi, row, col);
  int v;
  if (pi.fmt == FMT_I8A8) v = int(int8_t(code));
  else if (pi.asym) v = int(code) - int((blob + pi.zero_off)[mi]);
  else v = int(code) - pi.zc;
  out[i] = int16_t(v);
  if (scale_out) {
    const int gsz = pi.gpt ? 128 / pi.gpt : k;
    if (col % gsz == 0) {
      const size_t ci = pi.gpt ? size_t(row) * (k / gsz) + col / gsz : size_t(row);
      scale_out[ci] = reinterpret_cast<const float*>(blob + pi.scale_off)[mi];
    }
  }
}

int32_t launch_unpack(const moqe_qmat& p, const PackedInfo& pi, int16_t* out, float* scale_out, hipStream_t st) {
  ProfileScope ps(MOQE_PK_OTHER, st);
  size_t nel = size_t(p.n) * p.k;
  hipLaunchKernelGGL(k_unpack, dim3(unsigned((nel + 255) / 256)), dim3(256), 0, st,
                     static_cast<const uint8_t*>(p.qdata), p.n, p.k, pi, out, scale_out);
  return check_launch("unpack_qmat");
}

// ---- per-row dynamic int8 quantization of the rows of one expert's bucket --------------------
// Row b of the bucket (b < rows of the bucket) is read from x (gathered through perm when given)
// and written, as int8 with its scale, at its bucket-order position.
//   a = max|x|, sx = a/127 (1 if a == 0), xq = clamp(rint(x / sx), -127, 127)   (fp32 IEEE)
// The quotient is the correctly rounded one: with y = 1 / sx correctly rounded, q = x y is within an ulp of it and q + (x - q sx) y, the rest
// exact, rounds to it (Markstein), where nothing over- or underflows; rows of extreme scale divide.
// A work-group takes row after row and keeps a row's 4 NV KiB (2048 NV columns) in registers between the maximum and the rounding (NV 0: rows longer than 20480 are read again).
// A row is a chain of bucket offsets, its place, its values and the maximum over the work-group: 108 rows of 4096 8.3 -> 6.9 us by events, 1800 of 32768 rows of 18944
// in the bucket 53 -> 26.
template <int NV>
__global__ __launch_bounds__(256) void k_act_quant(const uint16_t* __restrict__ x, int kdim, int T,
                                                    const int32_t* __restrict__ offsets, const int32_t* __restrict__ perm,
                                                    int expert, int8_t* __restrict__ out, float* __restrict__ scales) {
  __shared__ float sh[4];
  const int off = offsets[expert];
  const int rows = (offsets[expert + 1] - off) * T;
  for (int b = blockIdx.x; b < rows; b += gridDim.x) {       // uniform over the work-group
    const int slot = off + b / T, t = b % T;
    const size_t src = perm ? size_t(perm[slot]) * T + t : size_t(off) * T + b;
    const size_t dst = size_t(off) * T + b;
    const uint4* xr = reinterpret_cast<const uint4*>(x + src * kdim);         // rows are multiples of 256 bytes
    uint2* o = reinterpret_cast<uint2*>(out + dst * kdim);
    const int nv = kdim >> 3;
    float a = 0.f;
    auto look = [&](const uint4& v) {
      const uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        a = fmaxf(a, fabsf(__uint_as_float(w[j] << 16)));
        a = fmaxf(a, fabsf(__uint_as_float(w[j] & 0xffff0000u)));
      }
    };
    uint4 kept[NV > 0 ? NV : 1];
    if constexpr (NV > 0) {
#pragma unroll
      for (int i = 0; i < NV; ++i) {
        const int c = int(threadIdx.x) + i * 256;
        kept[i] = c < nv ? xr[c] : make_uint4(0u, 0u, 0u, 0u);
      }
#pragma unroll
      for (int i = 0; i < NV; ++i) look(kept[i]);
    } else {
      for (int c = threadIdx.x; c < nv; c += 256) look(xr[c]);
    }
    a = block_max_256(a, sh);
    const float sx = (a == 0.f) ? 1.0f : __fdiv_rn(a, 127.0f);
    if (threadIdx.x == 0) scales[dst] = sx;
    const float y = __fdiv_rn(1.0f, sx);
    const bool plain = sx > 1e-30f && sx < 1e30f;            // uniform
    auto clamped = [](float q) { return uint32_t(uint8_t(int8_t(int(fminf(fmaxf(rintf(q), -127.f), 127.f))))); };
    if (!plain) {                                            // one element at a time: rare, and code that is not there need not be fetched
      const uint16_t* xs = x + src * kdim;
#pragma unroll 1
      for (int c = threadIdx.x; c < kdim; c += 256) out[dst * kdim + c] = int8_t(clamped(__fdiv_rn(__uint_as_float(uint32_t(xs[c]) << 16), sx)));
      continue;
    }
    auto code = [&](float v) {
      const float q = v * y;
      return clamped(fmaf(fmaf(-q, sx, v), y, q));
    };
    auto codes = [&](const uint4& v) {
      const uint32_t w[4] = {v.x, v.y, v.z, v.w};
      uint32_t h[4];
#pragma unroll
      for (int j = 0; j < 4; ++j) h[j] = code(__uint_as_float(w[j] << 16)) | code(__uint_as_float(w[j] & 0xffff0000u)) << 8;
      return make_uint2(h[0] | h[1] << 16, h[2] | h[3] << 16);
    };
    if constexpr (NV > 0) {
#pragma unroll
      for (int i = 0; i < NV; ++i) {
        const int c = int(threadIdx.x) + i * 256;
        if (c < nv) o[c] = codes(kept[i]);
      }
    } else {
      for (int c = threadIdx.x; c < nv; c += 256) o[c] = codes(xr[c]);
    }
  }
}

int32_t launch_act_quant(const void* x_bf16, int kdim, int T, const int32_t* offsets, const int32_t* perm,
                         int expert, int max_rows, int8_t* out, float* scales, hipStream_t st) {
  if (max_rows <= 0) return MOQE_OK;
  ProfileScope ps(MOQE_PK_ACTQUANT, st);
  // Up to 2048 work-groups, eight to a CU: the bucket's rows are known on the device only, and a launch of one for every row of the batch is mostly empty ones.
  auto go = [&](auto kernel) {
    hipLaunchKernelGGL(kernel, dim3(unsigned(max_rows < 2048 ? max_rows : 2048)), dim3(256), 0, st, static_cast<const uint16_t*>(x_bf16), kdim, T, offsets, perm, expert, out,
                       scales);
  };
  if (kdim <= 4096) go(k_act_quant<2>);
  else if (kdim <= 12288) go(k_act_quant<6>);
  else if (kdim <= 20480) go(k_act_quant<10>);
  else go(k_act_quant<0>);
  return check_launch("act_quant");
}

}  // namespace moqe
