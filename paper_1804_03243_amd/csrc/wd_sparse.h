// The sparse pruning sweep's choice of utterances and its search for a state
// among a frame's nodes, shared by the sweep and the link kernels.
#pragma once

#include "../../include/wfstdec.h"
#include "wd_block.h"

namespace wd {

// One frame's states as a search index in LDS: every 2^k-th of its n states
// from node n0 on.
struct SpFrame {
  uint64_t n0;
  uint32_t n, m, k;  // nodes, samples, stride as a shift
};

__device__ __forceinline__ SpFrame sp_frame(const LaneDesc& L, int t, uint32_t win) {
  SpFrame f;
  f.n0 = t >= 0 ? L.node_off[t] : 0;
  f.n = t >= 0 ? (uint32_t)(L.node_off[t + 1] - f.n0) : 0u;
  f.k = 0;
  while (((f.n + (1u << f.k) - 1u) >> f.k) > win) ++f.k;
  f.m = (f.n + (1u << f.k) - 1u) >> f.k;
  return f;
}

// The node of state s in frame f (~0 when it has none).
template <uint32_t WIN>
__device__ __forceinline__ uint32_t sp_lookup(const LaneDesc& L, const SpFrame& f, const uint32_t* win, uint32_t s) {
  if (f.m == 0 || win[0] > s) return ~0u;
  uint32_t i = 0;
#pragma unroll
  for (uint32_t step = WIN / 2; step; step >>= 1) {
    const uint32_t j = i + step;
    if (j < f.m && win[j] <= s) i = j;
  }
  if (f.k == 0) return win[i] == s ? (uint32_t)(f.n0 + i) : ~0u;
  uint32_t lo = i << f.k, hi = lo + (1u << f.k);
  hi = hi < f.n ? hi : f.n;
  while (hi - lo > 1u) {
    const uint32_t mid = (lo + hi) >> 1;
    if (L.n_state[f.n0 + mid] <= s) lo = mid;
    else hi = mid;
  }
  return L.n_state[f.n0 + lo] == s ? (uint32_t)(f.n0 + lo) : ~0u;
}

// Whether the pruning sweep of a finished utterance takes the sparse way: in
// one-workgroup mode from kSpTokens tokens a frame on (`chip`: always).  A
// sparse frame costs about 6 µs however many tokens it has; the dense sweep
// and link kernels cost 0.9 µs at 100 tokens and 75 µs at 7000.
constexpr uint64_t kSpTokens = 600;
__device__ __forceinline__ bool sparse_lane(const LaneDesc& L, uint32_t flags) {
  const LaneInfo* I = L.info;
  if (I->status != 0 || (I->overflow & kOvfNodes) || (flags & (WD_FLAG_DEBUG | WD_FLAG_NO_INCREMENTAL_PRUNE)))
    return false;
  return (flags & kFlagSwept) != 0 || I->tokens > kSpTokens * ((uint64_t)L.T + 1);
}

}  // namespace wd
