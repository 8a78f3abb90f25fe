// Small per-decode kernels around the decoder: input checks, fills, the lane
// frame ranges of a stream, and the packing of results for the host.
#include <algorithm>

#include "wd_cluster.h"
#include "wd_host.h"

namespace wd {

// Log-likelihood check: NaN, +inf and values above 1e30 are rejected.
// Rows of the frames this launch decodes, t0..T (frame t reads row t - 1).
// A streaming read: four independent loads per thread per step keep enough
// of them in flight to run at HBM speed.
__device__ __forceinline__ bool bad_loglike(float v) { return v != v || v > 1e30f; }

__global__ void k_check_loglikes(const LaneDesc* __restrict__ lanes, uint32_t P, uint32_t* bad) {
  const LaneDesc L = lanes[blockIdx.y];
  const uint64_t n = (uint64_t)L.T * P;
  const uint64_t r0 = (uint64_t)(L.t0 > 0 ? L.t0 - 1 : 0) * P;
  const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
  uint64_t i = r0 + (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
  bool b = false;
  for (; i + 3 * stride < n; i += 4 * stride) {
    const float v0 = L.ll[i], v1 = L.ll[i + stride], v2 = L.ll[i + 2 * stride], v3 = L.ll[i + 3 * stride];
    b |= bad_loglike(v0) | bad_loglike(v1) | bad_loglike(v2) | bad_loglike(v3);
  }
  for (; i < n; i += stride) b |= bad_loglike(L.ll[i]);
  if (b) atomicOr(&bad[blockIdx.y], 1u);
}

// Results of every finished utterance (links, nodes, words) packed into one
// contiguous buffer, so that the host copies them with one transfer: lane b
// starts after the lanes before it, each lane's part is its links, its nodes
// and its words padded to 16 bytes (packed_bytes; the host computes the same
// offsets).  One workgroup per lane.
__device__ __forceinline__ uint64_t packed_bytes(const LaneInfo& I) {
  if (I.status != 0 || I.tb_fail) return 0;
  return sizeof(OutLink) * I.kept + sizeof(OutNode) * I.out_nodes + ((4 * I.nwords + 15) & ~15ull);
}

__global__ void k_pack_results(const LaneDesc* __restrict__ lanes, int B, char* __restrict__ dst) {
  const int b = blockIdx.x;
  uint64_t off = 0;
  for (int k = 0; k < b; ++k) off += packed_bytes(*lanes[k].info);
  const LaneDesc& L = lanes[b];
  const LaneInfo& I = *L.info;
  if (!packed_bytes(I)) return;
  uint4* out = reinterpret_cast<uint4*>(dst + off);
  const uint64_t nl = I.kept * (sizeof(OutLink) / 16), nn = I.out_nodes;
  const uint4* ls = reinterpret_cast<const uint4*>(L.out_links);
  const uint4* ns = reinterpret_cast<const uint4*>(L.out_nodes);
  for (uint64_t i = threadIdx.x; i < nl; i += blockDim.x) out[i] = ls[i];
  for (uint64_t i = threadIdx.x; i < nn; i += blockDim.x) out[nl + i] = ns[i];
  uint32_t* w = reinterpret_cast<uint32_t*>(out + nl + nn);
  for (uint64_t i = threadIdx.x; i < I.nwords; i += blockDim.x) w[i] = (uint32_t)L.out_words[i];
}

void launch_pack_results(const LaneDesc* lanes, int B, void* dst, hipStream_t s) {
  hipLaunchKernelGGL(k_pack_results, dim3(B), dim3(256), 0, s, lanes, B, (char*)dst);
}

constexpr int kSetLanes = 128;
struct FrameSet {
  int32_t T[kSetLanes];
  int32_t t0[kSetLanes];
  int32_t b0, n, open;
};

// The headers of a cluster's control block, clean for a launch of the forward
// pass and of the pruning sweep.
__device__ __forceinline__ void clear_cluster(const LaneDesc& L) {
  WD_GLOBAL uint32_t* w = (WD_GLOBAL uint32_t*)L.ctl;
  if (!w) return;
  for (uint32_t i = threadIdx.x; i < kCtlHead / 4u; i += blockDim.x) {
    w[i] = 0;
    w[sizeof(ClusterCtl) / 4u + i] = 0;
  }
}

// A workgroup per utterance.
__global__ void k_set_frames(LaneDesc* lanes, FrameSet f) {
  LaneDesc& L = lanes[f.b0 + (int)blockIdx.x];
  if (threadIdx.x == 0) {
    L.T = f.T[blockIdx.x];
    L.t0 = f.t0[blockIdx.x];
    L.open = f.open;
  }
  clear_cluster(L);
}

// Everything a decode reads before writing, in one launch: the utterance's
// counters, its node bitmap and cluster headers; with `fill`, its slots and
// state bitmap too.
__global__ void __launch_bounds__(256) k_setup(const LaneDesc* __restrict__ lanes, uint32_t* bad, uint64_t used_words,
                                               uint64_t S, uint64_t bitmap_words, bool fill) {
  const LaneDesc& L = lanes[blockIdx.y];
  const uint64_t i0 = (uint64_t)blockIdx.x * 256 + threadIdx.x, step = (uint64_t)gridDim.x * 256;
  const uint64_t sum_words = L.slot2 && fill ? (bitmap_words + 31) / 32 : 0;
  for (uint64_t i = i0; i < used_words; i += step) L.used[i] = 0;
  if (fill) {
    for (uint64_t i = i0; i < S; i += step) {
      L.slot[i] = kEmpty;
      if (L.slot2) L.slot2[i] = kEmpty;
    }
    for (uint64_t i = i0; i < bitmap_words; i += step) L.bitmap[i] = 0;
    // (the bitmap's summary, where it has room: large frames keep it there)
    for (uint64_t i = i0; i < sum_words && i < L.frame_cap; i += step) L.surv_state[i] = 0;
  }
  if (blockIdx.x != 0) return;
  WD_GLOBAL uint32_t* info = (WD_GLOBAL uint32_t*)L.info;
  for (uint32_t i = threadIdx.x; i < sizeof(LaneInfo) / 4u; i += 256)
    info[i] = i == offsetof(LaneInfo, slots_clean) / 4u && fill ? 1u : 0u;
  if (threadIdx.x == 0) bad[blockIdx.y] = 0;
  clear_cluster(L);
}

// One-workgroup mode empties an utterance's slots (16 bytes per state) here for
// up to kFillLanes utterances, and otherwise in the utterance's first large
// frame, if it has one.  The chip empties 4.5 TB/s, the frame's workgroup 90 GB/s
// when no helper is up: one utterance on 30M states with three large frames
// spent 5.6 of 20.6 ms on that and spends 0.11 ms here, while 256 utterances on
// 5M states would spend 5 of 26 ms here.  The fill of some 50 utterances takes as long
// as a frame's own emptying; the line lies where it costs half of that, since in a
// batch of long utterances some frame usually is large, after the helpers have left
// (16 clean utterances of 500 frames on 5M states: 6.6 ms emptied by the frame,
// 5.8 ms here).
constexpr int kFillLanes = 24;

void launch_setup(const LaneDesc* lanes, int B, uint32_t* bad, uint64_t used_words, uint64_t S, uint64_t bitmap_words,
                  bool chip, hipStream_t s) {
  const bool fill = chip || B <= kFillLanes;
  const uint64_t n = fill ? std::max(used_words, S) : used_words;
  const uint64_t gx = std::min<uint64_t>(std::max<uint64_t>((n + 1023) / 1024, 1), B >= 64 ? 16 : 2048 / B);
  hipLaunchKernelGGL(k_setup, dim3((uint32_t)gx, B), dim3(256), 0, s, lanes, bad, used_words, S, bitmap_words, fill);
}

void launch_set_frames(LaneDesc* lanes, int B, const int32_t* T, const int32_t* t0, int32_t open, hipStream_t s) {
  for (int b0 = 0; b0 < B; b0 += kSetLanes) {
    FrameSet f{};
    f.b0 = b0;
    f.n = B - b0 < kSetLanes ? B - b0 : kSetLanes;
    f.open = open;
    for (int i = 0; i < f.n; ++i) {
      f.T[i] = T[b0 + i];
      f.t0[i] = t0[b0 + i];
    }
    hipLaunchKernelGGL(k_set_frames, dim3(f.n), dim3(128), 0, s, lanes, f);
  }
}


void launch_check_loglikes(const LaneDesc* lanes, int B, uint32_t P, uint32_t* bad, hipStream_t s) {
  // ~2048 workgroups in all (at least 16 per utterance)
  const int gx = B >= 128 ? 16 : 2048 / B;
  hipLaunchKernelGGL(k_check_loglikes, dim3(gx, B), dim3(256), 0, s, lanes, P, bad);
}

}  // namespace wd
