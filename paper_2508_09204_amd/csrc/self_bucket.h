// Device-side bucketing of at most 64 samples inside a grouped launch (GemmArgs::expert_idx), shared by the streaming kernels.
#pragma once

#include "moqe_internal.h"

namespace moqe {

// Stable counting sort, a sample per lane: the count of expert k is the population of the ballot "my sample goes to k", a sample's place in
// its bucket the population below its lane (the bucket kernel's arithmetic).  Lanes whose `e` is an expert leave with its
// bounds o0 .. o1; perm_l (64 entries, this wave's own) gets the permutation; with `publish` (one wave of the launch) counts, offsets
// and permutations go to memory for the launches after it.  Must be called by whole waves.
static __device__ __forceinline__ void self_bucket(const GemmArgs& ga, const int e, int& o0, int& o1, int32_t* perm_l, const bool publish) {
  const int K = ga.n_experts, L = threadIdx.x & 63;
  int es = L < ga.S ? ga.expert_idx[L] : -1;
  if (es >= K) es = -1;
  const unsigned long long below = L == 0 ? 0ull : (~0ull >> (64 - L));
  int base = 0, my_pos = 0;
  o0 = 0; o1 = 0;
  for (int k = 0; k < K; ++k) {
    const unsigned long long b = __ballot(es == k);
    const int c = __popcll(b);
    if (es == k) my_pos = base + __popcll(b & below);
    if (e == k) { o0 = base; o1 = base + c; }
    base += c;
  }
  if (es >= 0) perm_l[my_pos] = L;                      // this wave's own copy: read back by the same wave only
  __builtin_amdgcn_wave_barrier();
  if (publish) {
    if (L < K) {
      if (ga.out_counts) ga.out_counts[L] = o1 - o0;
      if (ga.out_offsets) ga.out_offsets[L] = o0;
    }
    if (L == 0 && ga.out_offsets) ga.out_offsets[K] = base;
    if (es >= 0) {
      if (ga.out_perm) ga.out_perm[my_pos] = L;
      if (ga.out_inv_perm) ga.out_inv_perm[L] = my_pos;
    }
  }
}

}  // namespace moqe
