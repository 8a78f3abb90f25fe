// Large frames of the one-workgroup forward pass, shared by a cluster of
// workgroups on one XCD.
//
// A frame that outgrows the LDS token table (thousands of tokens: flat
// log-likelihoods, where max-active is what limits a frame) is tens of
// thousands of independent random accesses, which one CU cannot keep in
// flight.  The utterance's workgroup (the leader) then runs the frame together
// with helper workgroups that the same launch put on the leader's XCD.  All of
// them reach the same L2, so what they share needs no write-back: stores end
// in the L2 (s_waitcnt vmcnt(0) before a cluster barrier), and every read of
// shared data is a device-scope load, which passes the CU's own L1.  A barrier
// of 31 workgroups measured 1.0 µs this way (2.8 µs with an L1 invalidation
// per workgroup, 29 µs with one per wavefront; a kernel launch per step costs
// ~4.6 µs, and steps of a 7000-token frame take 1-3 µs each).
//
// Nothing waits for a workgroup that may not be running: helpers register for
// a run of frames while the leader holds the registration open for a few
// microseconds, and the barriers count the registered ones only.  A helper
// that is idle for kIdleTicks (and a quarter of the time it has worked) leaves,
// so the CUs of utterances that never have a large frame are free for other
// work soon after the launch; in a launch that resumes parked utterances, which
// have such frames, it stays for kIdleResumed.
//
// Per frame t, with the tokens of frame t - 1 as bits of a state bitmap (and
// their packed tokens in the slot array of that frame's parity):
//   A  each workgroup takes a contiguous range of the kept tokens (equal
//      shares, found from counts per 2048 state ranges), numbers them in
//      state order, stores them as nodes and frontier, and expands its own
//      tokens' emitting arcs into frame t's slot array: no prefix sum over the
//      cluster, no exchange of the frontier;
//   B  the epsilon closure: every epsilon path of the bucketed states within
//      the cutoff (level by level without a path table);
//   C  survivors of the beam cutoff, and the histogram for max-active;
//   D  further digits of the max-active radix select, when it binds;
//   E  kept tokens into the bitmap (in C when max-active cannot bind).
// Results are those of the LDS path bit for bit: the same sums, the same
// minima, the same cutoffs.
#pragma once

#include <stddef.h>

#include "wd_block.h"
#include "wd_spin.h"

namespace wd {

constexpr uint32_t kXcds = 8;              // consecutive workgroups go to the XCDs in turn
constexpr uint32_t kClMax = 32;            // workgroups of a cluster (an XCD has 32 CUs)
constexpr uint32_t kCoarse = 2048;         // state ranges counted for the shares of phase A
constexpr uint32_t kClDigits = 3;          // radix digits of a 32-bit key (11, 11, 10)
constexpr uint64_t kIdleTicks = 30000;     // 300 µs of the 100 MHz clock
// helpers of utterances known to have large frames: 2 ms, some 250 small frames
constexpr uint64_t kIdleResumed = 200000;
constexpr uint64_t kJoinTicks = 400;       // a run waits for its helpers this long at most (4 µs)
constexpr uint32_t kRegroupFrames = 4;     // frames after which a run takes in late helpers
// back to the LDS path once a frame is this small
constexpr uint32_t kSmallTokens = 512;
constexpr uint32_t kSmallTouched = 1400;

// Shared control block of one utterance's cluster (workspace; zeroed up to
// `f` before every launch).
struct alignas(128) ClusterCtl {
  uint32_t xcc;     // the leader's XCD + 1, 0 until it runs
  uint32_t cmd;     // number of the run the leader last opened
  uint32_t quit;    // the leader is done
  uint32_t bad;     // a wait ran into its limit
  uint32_t pad0[28];
  uint32_t tickets; // helpers that have come up
  uint32_t alive;   // of them, not gone
  uint32_t pad1[30];
  uint32_t join[kClMax];    // per helper: the run it waits to be taken into
  unsigned long long members;  // run << 32 | mask of the helpers in it
  uint32_t t;       // the run's first frame
  uint32_t n_prev;  // tokens of the frame before it
  uint32_t node_base;  // nodes before that frame's successor (low, high)
  uint32_t node_base_hi;
  uint32_t clear;   // the slot arrays have to be emptied first
  uint32_t hist_ok;
  uint32_t bar0;    // barrier arrivals before the run
  uint32_t pad3;
  unsigned long long links;  // raw lattice links of the run's frames
  uint32_t pad4[20];
  uint32_t bar;     // barrier arrivals
  uint32_t pad5[31];
  struct alignas(128) Frame {
    uint32_t best;       // smallest emitting candidate key, inverted (so that 0 is "none")
    uint32_t n_touched;
    uint32_t n_bk;       // bucketed by the expansion
    uint32_t n_bx;       // reached by epsilon paths (bucketed by level without a path table)
    uint32_t n_surv;
    uint32_t regroup;    // helpers wait for the next run: the leader ends this one
    uint32_t pad0[2];
    unsigned long long work;  // emitting arcs
    unsigned long long eps;   // epsilon arcs of the closure
    uint32_t pad1[20];
  } f[2];
  uint32_t coarse[2][kCoarse];
  uint32_t hist[kClDigits][kHistBins];
};

// What a run of large frames leaves for the leader.
struct ClusterState {
  int t;               // first frame not done
  int status;
  uint32_t ovf;
  uint32_t n_prev, W;  // tokens of the last frame done, their emitting arcs
  uint32_t hist_ok;
  uint32_t again;      // the next frame is to be run as a large one, too
  uint64_t node_base;  // nodes before frame t
  uint64_t arcs, eps, links, tokens, max_tokens, need_frame, need_arcs;  // of the run's frames
};

// The pruning sweep's cluster has a header of its own behind the block (of a
// ClusterCtl only the part before `f`), so that it finds it clean.
constexpr size_t kCtlHead = offsetof(ClusterCtl, f);
constexpr size_t kCtlBytes = sizeof(ClusterCtl) + kCtlHead;

// LDS of a workgroup while it runs large frames (laid over the LDS path's
// token table and frontier).
constexpr uint32_t kClTile = 1024;   // tokens or bucket entries per tile
constexpr uint32_t kClRounds = 4;    // rounds of one touch per thread before the stage is flushed
constexpr uint32_t kHeld = 3;        // touched states a thread keeps in registers over a frame's last steps
constexpr uint32_t kSumList = 4096;  // bitmap words listed at once (in the stage)
constexpr uint32_t kClBk = 2048;     // states with epsilon arcs staged
constexpr uint32_t kClCand = 12288;  // candidate cost keys a workgroup keeps for the link count
struct ClusterShared {
  BlockScratch bs;
  uint32_t pre[kClTile], beg[kClTile], key[kClTile], xbeg[kClTile], deg[kClTile];
  uint32_t cand[kClCand];
  uint32_t st_n, st_nb, st_at, st_bat, n_cand;
  uint32_t st[kClRounds * kThreads];
  uint4 bk[kClBk];
  uint32_t hist[kHistBins];
  uint32_t sel[4];
  uint32_t lo, hi, base;  // this workgroup's state ranges, its first token
  uint32_t go;
  ClusterState out;
};
static_assert(kSumList <= kClRounds * (uint32_t)kThreads, "listed bitmap words in the stage");
static_assert(kClTile == (uint32_t)kThreads, "one token or entry of a tile per thread");

// ------------------------------------------------------------ shared memory

template <class T>
__device__ __forceinline__ T cl_load(const WD_GLOBAL T* p) {
  return __hip_atomic_load(const_cast<WD_GLOBAL T*>(p), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
template <class T>
__device__ __forceinline__ void cl_store(WD_GLOBAL T* p, T v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
template <class T>
__device__ __forceinline__ T cl_add(WD_GLOBAL T* p, T v) {
  return __hip_atomic_fetch_add(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Every store of this wavefront has reached the L2.
__device__ __forceinline__ void cl_drain() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }

// XCD this workgroup runs on (hardware register XCC_ID).
__device__ __forceinline__ uint32_t cl_xcc() { return (uint32_t)__builtin_amdgcn_s_getreg(20 | (3 << 11)) & 15u; }

typedef WD_GLOBAL ClusterCtl Ctl;
typedef WD_GLOBAL ClusterCtl::Frame CtlFrame;

// Barrier over the run's N workgroups.  `gen` is the arrivals that complete
// the last one, the same in every thread; the count runs on over the runs of a
// launch, so that a workgroup still leaving a run's last barrier is not caught
// by the next run.  A wait beyond its limit marks the run bad; the callers
// stop at the next check.
__device__ __forceinline__ void cl_barrier(Ctl* C, uint32_t N, uint32_t& gen) {
  gen += N;
  cl_drain();
  __syncthreads();
  if (N > 1u) {
    if (threadIdx.x == 0) {
      cl_add<uint32_t>(&C->bar, 1u);
      const uint32_t target = gen;
      if (!arrived(cl_load(&C->bar), target)) {
        SpinClock spin(wall_clock64());
        for (uint32_t n = 1; !arrived(cl_load(&C->bar), target); ++n)
          if (n % kSpinLooks == 0 && spin.beyond(wall_clock64())) {
            cl_store(&C->bad, 1u);
            break;
          }
      }
    }
    __syncthreads();
  }
}

// Last i in [0, n) with a[i] <= w, in LDS (a non-decreasing, a[0] <= w, n <= kClTile).
__device__ __forceinline__ uint32_t cl_find(const uint32_t* a, uint32_t n, uint32_t w) {
  uint32_t i = 0;
#pragma unroll
  for (uint32_t step = kClTile / 2; step; step >>= 1) {
    const uint32_t j = i + step;
    i = j < n && a[j] <= w ? j : i;
  }
  return i;
}

// First touches of a state: staged in LDS by whole wavefronts, appended to
// the frame's lists with one add per list and flush.  kRounds rounds of one
// touch per thread fit the stage; states with epsilon arcs beyond kClBk are
// appended one by one.
// Bucketed states: with a path table {state, its paths, its epsilon degree}
// (the expansion's; what paths reach goes to the level lists' arrays); level by
// level {state, level} in f_xbeg / f_xdeg, which hold a frame's touched states.
__device__ __forceinline__ void cl_bucket_level(CtlFrame* F, const LaneDesc& L, uint32_t state, uint32_t v) {
  const uint32_t q = cl_add<uint32_t>(&F->n_bx, 1u);
  if (q < L.frame_cap) {
    L.f_xbeg[q] = state;
    L.f_xdeg[q] = v;
  }
}
__device__ __forceinline__ void cl_bucket_path(CtlFrame* F, const LaneDesc& L, uint4 e) {
  const uint32_t q = cl_add<uint32_t>(&F->n_bk, 1u);
  if (q < L.cand_cap) L.cand[q] = e;
}

__device__ __forceinline__ void cl_flush(ClusterShared& S, CtlFrame* F, const LaneDesc& L, bool paths) {
  __syncthreads();
  const uint32_t n = S.st_n, nb = S.st_nb < kClBk ? S.st_nb : kClBk;
  if (threadIdx.x == 0 && n) S.st_at = cl_add<uint32_t>(&F->n_touched, n);
  if (threadIdx.x == 64 && nb) S.st_bat = cl_add<uint32_t>(paths ? &F->n_bk : &F->n_bx, nb);
  __syncthreads();
  for (uint32_t i = threadIdx.x; i < n; i += kThreads)
    if ((uint64_t)S.st_at + i < L.frame_cap) L.touched[S.st_at + i] = S.st[i];
  for (uint32_t i = threadIdx.x; i < nb; i += kThreads) {
    const uint64_t q = (uint64_t)S.st_bat + i;
    const uint4 e = S.bk[i];
    if (paths) {
      if (q < L.cand_cap) L.cand[q] = e;
    } else if (q < L.frame_cap) {
      L.f_xbeg[q] = e.x;
      L.f_xdeg[q] = e.w;
    }
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    S.st_n = 0;
    S.st_nb = 0;
  }
  __syncthreads();
}

__device__ __forceinline__ uint4 cl_load4(const WD_GLOBAL uint4* p) {
  const WD_GLOBAL unsigned long long* q = (const WD_GLOBAL unsigned long long*)p;
  const unsigned long long a = cl_load(q), b = cl_load(q + 1);
  return make_uint4((uint32_t)a, (uint32_t)(a >> 32), (uint32_t)b, (uint32_t)(b >> 32));
}

__device__ __forceinline__ unsigned long long cl_min64(WD_GLOBAL unsigned long long* p, unsigned long long v) {
  return __hip_atomic_fetch_min(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// A kept token of state s: its bit (with `sum`: and the bit of its bitmap word
// in the summary, kept in surv_state, which large frames do not need), and its
// range's count.
__device__ __forceinline__ void cl_mark(Ctl* C, const LaneDesc& L, bool sum, int t, uint32_t wsh, uint32_t s) {
  (void)__hip_atomic_fetch_or(&L.bitmap[s >> 5], 1u << (s & 31u), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  if (sum)
    (void)__hip_atomic_fetch_or(&L.surv_state[s >> 10], 1u << ((s >> 5) & 31u), __ATOMIC_RELAXED,
                                __HIP_MEMORY_SCOPE_AGENT);
  cl_add<uint32_t>(&C->coarse[t & 1][s >> (5u + wsh)], 1u);
}

// The bin of a histogram (shared by the cluster) that holds the rank-th
// smallest key; whole workgroup.
__device__ __forceinline__ void cl_select_bin(const WD_GLOBAL uint32_t* hist, uint32_t rank, ClusterShared& S,
                                              uint32_t& par, uint32_t* bin, uint32_t* before, uint32_t* count) {
  const uint32_t tid = threadIdx.x;
  const uint32_t h0 = cl_load(&hist[2 * tid]), h1 = cl_load(&hist[2 * tid + 1]);
  uint32_t tot;
  const uint32_t ex = block_excl_scan(h0 + h1, S.bs, par, &tot);
  if (ex < rank && rank <= ex + h0) {
    S.sel[0] = 2 * tid;
    S.sel[1] = ex;
    S.sel[2] = h0;
  } else if (ex + h0 < rank && rank <= ex + h0 + h1) {
    S.sel[0] = 2 * tid + 1;
    S.sel[1] = ex + h0;
    S.sel[2] = h1;
  }
  __syncthreads();
  *bin = S.sel[0];
  *before = S.sel[1];
  *count = S.sel[2];
  __syncthreads();
}

// Adds the workgroup's LDS histogram to the cluster's and empties it.
__device__ __forceinline__ void cl_merge_hist(ClusterShared& S, WD_GLOBAL uint32_t* hist) {
  __syncthreads();
  for (uint32_t i = threadIdx.x; i < (uint32_t)kHistBins; i += kThreads) {
    const uint32_t v = S.hist[i];
    if (v) {
      cl_add<uint32_t>(&hist[i], v);
      S.hist[i] = 0;
    }
  }
}

// One run of large frames, from frame C->t on: workgroup w of N.  Ends after
// a small frame, after the last frame, or with a status; the leader (w = 0)
// finds the outcome in S.out.
__device__ __forceinline__ void cl_run(const DevGraph& g, const LaneDesc& L, const Params& prm, ClusterShared& S,
                                       Ctl* C, uint32_t w, uint32_t N, bool paths) {
  const uint32_t tid = opaque(threadIdx.x);  // (nothing of a run is held across the LDS frames)
  const int T = L.T;
  uint32_t par = 0, gen = cl_load(&C->bar0);
  int t = (int)cl_load(&C->t);
  uint32_t n_all = cl_load(&C->n_prev);
  uint64_t nb = ((uint64_t)cl_load(&C->node_base_hi) << 32) | cl_load(&C->node_base);  // nodes before frame t
  bool hist_ok = cl_load(&C->hist_ok) != 0;
  const uint32_t nw = (g.S + 31u) >> 5;
  uint32_t wsh = 0;  // bitmap words per counted range, as a shift
  while ((nw >> wsh) >= kCoarse) ++wsh;
  // a summary bit per bitmap word, where there is room for it and a counted
  // range is whole summary words (so that no two workgroups share one)
  const bool sum = wsh >= 5u && (uint64_t)L.frame_cap * 32u >= nw;
  // ------------------------------------------------ a clean control block
  if (cl_load(&C->clear)) {
    const uint64_t n = (uint64_t)g.S, lo = n * w / N, hi = n * (w + 1) / N;
    for (uint64_t i = lo + tid; i < hi; i += kThreads) {
      L.slot[i] = kEmpty;
      L.slot2[i] = kEmpty;
    }
    for (uint32_t i = w * kThreads + tid; i < nw; i += N * kThreads) L.bitmap[i] = 0;
    if (sum)
      for (uint32_t i = w * kThreads + tid; i < (nw + 31u) >> 5; i += N * kThreads) L.surv_state[i] = 0;
  }
  for (uint32_t i = w * kThreads + tid; i < kCoarse; i += N * kThreads) {
    C->coarse[0][i] = 0;
    C->coarse[1][i] = 0;
  }
  for (uint32_t i = w * kThreads + tid; i < kClDigits * kHistBins; i += N * kThreads) (&C->hist[0][0])[i] = 0;
  if (w == 0 && tid < 2u * sizeof(ClusterCtl::Frame) / 4u) ((WD_GLOBAL uint32_t*)&C->f[0])[tid] = 0;
  for (uint32_t i = tid; i < (uint32_t)kHistBins; i += kThreads) S.hist[i] = 0;
  if (tid == 0) {
    S.st_n = 0;
    S.st_nb = 0;
    S.out = ClusterState{};
  }
  if (w == 0 && tid == 0) cl_store<unsigned long long>(&C->links, 0ull);
  cl_barrier(C, N, gen);

  uint64_t my_links = 0;  // raw lattice links found by this thread
  bool stored = true;  // the frontier of frame t - 1 is in the workspace, with degree prefix sums
  bool small = false;  // frame t - 1 touched few states
  bool regroup = false;  // the run ends so that more helpers can join the next
  uint32_t frames = 0;
  uint32_t best_key = 0, kcutb = 0, cut_key = 0;  // of frame t - 1 (from the second frame on)
  int status = 0;
  uint32_t ovf = 0;
  auto stamp = [&](int f, int k) {
    if (L.prof && w == 0 && tid == 0) L.prof[(size_t)f * kProfSlots + (size_t)k] = wall_clock64();
  };
  while (true) {
    // ---------------------------- A: tokens of frame t - 1, expansion of frame t
    WD_GLOBAL unsigned long long* const cur = (t & 1) ? L.slot2 : L.slot;
    WD_GLOBAL unsigned long long* const prev = (t & 1) ? L.slot : L.slot2;
    CtlFrame* const F = &C->f[t & 1];
    uint32_t n0, n1;
    bool done = false;
    if (stored) {
      n0 = (uint32_t)((uint64_t)n_all * w / N);
      n1 = (uint32_t)((uint64_t)n_all * (w + 1) / N);
    } else {
      // equal shares of the kept tokens, cut at the counted ranges: from the
      // first range that starts at or after the share's first token on
      const WD_GLOBAL uint32_t* co = C->coarse[(t - 1) & 1];
      const uint32_t c0 = cl_load(&co[2 * tid]), c1 = cl_load(&co[2 * tid + 1]);
      const uint32_t ex = block_excl_scan(c0 + c1, S.bs, par, &n_all);
      S.hist[2 * tid] = ex;
      S.hist[2 * tid + 1] = ex + c0;
      if (tid == 0) {
        S.lo = S.hi = kCoarse;
        S.base = n_all;
      }
      __syncthreads();
      const uint32_t a = (uint32_t)((uint64_t)n_all * w / N), b = (uint32_t)((uint64_t)n_all * (w + 1) / N);
      for (uint32_t q = 2 * tid; q < 2 * tid + 2; ++q) {
        const uint32_t p = S.hist[q];
        const bool first = q == 0;
        const uint32_t before = first ? 0u : S.hist[q - 1];
        if (p >= a && (first || before < a)) {
          S.lo = q;
          S.base = p;
        }
        if (w + 1 < N && p >= b && (first || before < b)) S.hi = q;
      }
      __syncthreads();
      const uint32_t lo = S.lo, hi = S.hi;
      n0 = S.base;
      __syncthreads();
      S.hist[2 * tid] = 0;
      S.hist[2 * tid + 1] = 0;
      // the states, in order
      const uint32_t w0 = lo << wsh, w1 = (uint64_t)(hi << wsh) < nw ? hi << wsh : nw;
      n1 = n0;
      // the bits of word v (number i of the bitmap) from position p on
      auto spread = [&](uint32_t i, uint32_t v, uint32_t p) {
        if (v) L.bitmap[i] = 0;
        while (v) {
          const uint32_t bit = (uint32_t)__ffs(v) - 1u;
          v &= v - 1u;
          L.f_state[p++] = (i << 5) | bit;
        }
      };
      if (sum) {
        // the summary names the words that are not empty: they are listed in
        // LDS, then one word per thread (625 KB of bitmap at 5M states took 11
        // of a frame's 59 µs with 8 workgroups)
        for (uint32_t b = w0 >> 5; b < (w1 + 31u) >> 5; b += kThreads) {
          const uint32_t i = b + tid;
          const uint32_t v = i < (w1 + 31u) >> 5 ? cl_load(&L.surv_state[i]) : 0u;
          if (v) L.surv_state[i] = 0;
          uint32_t words;
          const uint32_t p0 = block_excl_scan((uint32_t)__popc(v), S.bs, par, &words);
          for (uint32_t c0 = 0; c0 < words; c0 += kSumList) {
            uint32_t p = p0 - c0;  // (mod 2^32: below or beyond this part of the list)
            for (uint32_t m = v; m; m &= m - 1u, ++p)
              if (p < kSumList) S.st[p] = (i << 5) | ((uint32_t)__ffs(m) - 1u);
            __syncthreads();
            const uint32_t n = words - c0 < kSumList ? words - c0 : kSumList;
            for (uint32_t c = 0; c < n; c += kThreads) {
              const bool on = c + tid < n;
              const uint32_t q = on ? S.st[c + tid] : 0u;
              const uint32_t word = on ? cl_load(&L.bitmap[q]) : 0u;
              uint32_t tot;
              const uint32_t at = n1 + block_excl_scan((uint32_t)__popc(word), S.bs, par, &tot);
              n1 += tot;
              spread(q, word, at);
            }
            __syncthreads();
          }
        }
      } else {
        for (uint32_t b = w0; b < w1; b += 4 * kThreads) {
          uint32_t word[4], c = 0;
#pragma unroll
          for (uint32_t k = 0; k < 4; ++k) {
            const uint32_t i = b + 4 * tid + k;
            word[k] = i < w1 ? cl_load(&L.bitmap[i]) : 0u;
            c += (uint32_t)__popc(word[k]);
          }
          uint32_t tot;
          uint32_t p = n1 + block_excl_scan(c, S.bs, par, &tot);
          n1 += tot;
#pragma unroll
          for (uint32_t k = 0; k < 4; ++k) {
            spread(b + 4 * tid + k, word[k], p);
            p += (uint32_t)__popc(word[k]);
          }
        }
      }
      cl_drain();
      __syncthreads();
      if (hist_ok && nb + n_all > L.node_cap) {
        hist_ok = false;
        ovf |= kOvfNodes;
      }
      if (w == 0 && tid == 0) {
        L.node_off[t - 1] = nb;
        L.node_off[t] = nb + n_all;
        L.best[t - 1] = key_cost(best_key);
        L.cutb[t - 1] = key_cost(kcutb);
        L.cut[t - 1] = key_cost(cut_key);
        L.xmask[t - 1] = 1;  // (the frame's raw links are counted here)
        S.out.tokens += n_all;
        if (n_all > S.out.max_tokens) S.out.max_tokens = n_all;
        if (L.prof) L.prof[(size_t)(t - 1) * kProfSlots + kProfStamps] = (uint64_t)n_all << 8;
      }
      for (int k = 6; k < kProfStamps; ++k) stamp(t - 1, k);
      done = t > T || regroup || (small && n_all <= kSmallTokens);
    }
    if (!done) stamp(t, 0);
    const float* row = (const float*)L.ll + (size_t)(t > 0 ? t - 1 : 0) * g.P;
    uint32_t my_best = 0xffffffffu;
    if (tid == 0) S.n_cand = 0;
    __syncthreads();
    if (t == 0 && w == 0) {  // the start token
      if (tid == 0) {
        const uint32_t s0 = g.start, cls = g.sclass[s0];
        cur[s0] = pack_tok(cost_key(0.0f), kNoArc);
        S.st[0] = s0;
        S.st_n = 1;
        if (cls != kNoEps) {
          const uint4 o0 = g.off[s0], o1 = g.off[s0 + 1];
          S.bk[0] = paths ? make_uint4(s0, o0.z, o1.z, o1.y - o0.y) : make_uint4(s0, 0, 0, cls);
          S.st_nb = 1;
        }
        my_best = cost_key(0.0f);
      }
      cl_flush(S, F, L, paths);
    }
    for (uint32_t tb = n0; tb < n1; tb += kClTile) {
      const uint32_t m = n1 - tb < kClTile ? n1 - tb : kClTile;
      uint32_t deg = 0, beg = 0, key = 0, xdeg = 0, xbeg = 0;
      if (tid < m) {
        const uint32_t p = tb + tid;
        if (stored) {
          key = cl_load(&L.f_key[p]);
          beg = cl_load(&L.f_ebeg[p]);
          deg = cl_load(&L.f_edeg[p + 1]) - cl_load(&L.f_edeg[p]);
        } else {
          const uint32_t s = cl_load(&L.f_state[p]);
          const unsigned long long v = cl_load(&prev[s]);
          const uint4 o0 = g.off[s], o1 = g.off[s + 1];
          prev[s] = kEmpty;
          key = (uint32_t)(v >> 32);
          beg = o0.x;
          deg = done ? 0u : o1.x - o0.x;
          xbeg = o0.y;
          xdeg = o1.y - o0.y;
          L.f_key[p] = key;
          if (hist_ok) {
            L.n_state[nb + p] = s;
            L.n_pack[nb + p] = v;
            L.n_pred[nb + p] = kNoArc;
          }
        }
      }
      // items: each token's emitting arcs, then its epsilon arcs (frame t - 1's
      // epsilon links, which are only counted)
      uint32_t tot;
      S.pre[tid] = block_excl_scan(deg + xdeg, S.bs, par, &tot);
      S.beg[tid] = beg;
      S.key[tid] = key;
      S.deg[tid] = deg;
      S.xbeg[tid] = xbeg;
      __syncthreads();
      // two items per thread at a time, each step's loads together
      constexpr uint32_t kU = 2;
      uint32_t round = 0;
      for (uint32_t b = 0; b < tot; b += kU * kThreads) {
        uint32_t j[kU];
        bool emit[kU], eps[kU], first[kU];
        uint4 r[kU];
        uint2 ox[kU], op[kU];  // a destination's epsilon degree's ends, its paths
#pragma unroll
        for (uint32_t u = 0; u < kU; ++u) {
          const uint32_t it = b + u * kThreads + tid;
          emit[u] = false;
          j[u] = 0;
          r[u] = make_uint4(0, kNoArc, 0, 0);
          if (it < tot) {
            j[u] = cl_find(S.pre, m, it);
            const uint32_t i = it - S.pre[j[u]], de = S.deg[j[u]];
            emit[u] = i < de;
            r[u] = emit[u] ? g.earc[S.beg[j[u]] + i] : g.xarc[S.xbeg[j[u]] + (i - de)];
          }
        }
        float ac[kU];
#pragma unroll
        for (uint32_t u = 0; u < kU; ++u) {
          eps[u] = emit[u] && (r[u].z >> 24) != kNoEps;
          ac[u] = emit[u] ? -row[(r[u].z & 0xffffffu) - 1u] : 0.0f;
          ox[u] = op[u] = make_uint2(0, 0);
          if (eps[u] && paths) {
            const uint4 o0 = g.off[r[u].x], o1 = g.off[r[u].x + 1];
            ox[u] = make_uint2(o0.y, o1.y);
            op[u] = make_uint2(o0.z, o1.z);
          }
        }
#pragma unroll
        for (uint32_t u = 0; u < kU; ++u) {
          const uint32_t at = wave_append(emit[u], &S.n_cand);
          first[u] = false;
          const float c = key_cost(S.key[j[u]]);
          if (emit[u]) {
            const float x = canon((c + ac[u]) + __uint_as_float(r[u].y));
            const uint32_t xk = cost_key(x);
            if (at < kClCand) S.cand[at] = xk;
            if (xk < kInfKey) {
              my_best = xk < my_best ? xk : my_best;
              first[u] = cl_min64(&cur[r[u].x], pack_tok(xk, r[u].w)) == kEmpty;
            }
          } else if (b + u * kThreads + tid < tot) {
            const uint32_t xk = cost_key(canon(c + __uint_as_float(r[u].y)));
            my_links += xk <= cut_key && xk < kInfKey ? 1u : 0u;
          }
        }
#pragma unroll
        for (uint32_t u = 0; u < kU; ++u) {
          const uint32_t p = wave_append(first[u], &S.st_n);
          if (first[u]) S.st[p] = r[u].x;
          const uint32_t q = wave_append(first[u] && eps[u], &S.st_nb);
          if (first[u] && eps[u]) {
            const uint4 e = paths ? make_uint4(r[u].x, op[u].x, op[u].y, ox[u].y - ox[u].x)
                                  : make_uint4(r[u].x, 0, 0, r[u].z >> 24);
            if (q < kClBk) S.bk[q] = e;
            else if (paths) cl_bucket_path(F, L, e);
            else cl_bucket_level(F, L, e.x, e.w);
          }
        }
        if (++round % (kClRounds / kU) == 0) cl_flush(S, F, L, paths);
      }
      cl_flush(S, F, L, paths);
    }
    if (!stored) nb += n_all;
    if (done) break;
    const uint32_t my_work = S.n_cand;  // this workgroup's emitting arcs
    my_best = (uint32_t)block_min64(my_best, S.bs, par);
    if (tid == 0) {
      if (my_best != 0xffffffffu)
        (void)__hip_atomic_fetch_max(&F->best, ~my_best, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      if (my_work) cl_add<unsigned long long>(&F->work, (unsigned long long)my_work);
    }
    stored = false;
    cl_barrier(C, N, gen);
    if (cl_load(&C->bad)) {
      status = kStatusInternal;
      break;
    }
    // ---------------------------------------------------- B: epsilon closure
    const uint64_t work = cl_load(&F->work);
    if (w == 0 && tid == 0) {
      if (work > S.out.need_arcs) S.out.need_arcs = work;
      if (L.prof) L.prof[(size_t)t * kProfSlots + kProfStamps + 1] = work | ((uint64_t)N << 32);
    }
    if (work > L.cand_cap) {
      status = 4;  // WD_ECAPACITY
      ovf |= kOvfArcs;
      break;
    }
    stamp(t, 1);
    best_key = ~cl_load(&F->best);
    if (best_key >= kInfKey) {
      status = 3;  // WD_ENOPATH
      break;
    }
    if (w == 0 && tid == 0) S.out.arcs += work;
    kcutb = cost_key(key_cost(best_key) + prm.beam);
    // the next frame's control block, and the histograms (last read before
    // the last barrier of frame t - 1)
    {
      CtlFrame* const F1 = &C->f[(t + 1) & 1];
      if (w == 0 && tid < sizeof(ClusterCtl::Frame) / 4u) ((WD_GLOBAL uint32_t*)F1)[tid] = 0;
      for (uint32_t i = w * kThreads + tid; i < kCoarse; i += N * kThreads) C->coarse[(t + 1) & 1][i] = 0;
      for (uint32_t i = w * kThreads + tid; i < kClDigits * kHistBins; i += N * kThreads) (&C->hist[0][0])[i] = 0;
    }
    // a path's or arc's result into its state; whole wavefronts
    auto relax = [&](bool on, uint32_t dst, uint32_t xk, uint32_t arc) -> bool {
      bool first = false;
      if (on && xk <= kcutb && xk < kInfKey) first = cl_min64(&cur[dst], pack_tok(xk, arc)) == kEmpty;
      const uint32_t p = wave_append(first, &S.st_n);
      if (first) S.st[p] = dst;
      return first;
    };
    const uint32_t nlev = paths ? 1u : g.nlevels;
    for (uint32_t lvl = 0; lvl < nlev; ++lvl) {
      // the entries there now (with paths the closure appends to the other
      // list; level by level the count is taken before anyone appends more,
      // and every entry of this level is there)
      uint32_t n_bk = paths ? cl_load(&F->n_bk) : cl_load(&F->n_bx);
      if (!paths) cl_barrier(C, N, gen);
      // (beyond the capacity: the frame is about to stop)
      const uint64_t cap = paths ? L.cand_cap : L.frame_cap;
      if (n_bk > cap) n_bk = (uint32_t)cap;
      const uint32_t e0 = (uint32_t)((uint64_t)n_bk * w / N), e1 = (uint32_t)((uint64_t)n_bk * (w + 1) / N);
      for (uint32_t tb = e0; tb < e1; tb += kClTile) {
        uint32_t d = 0, key = 0, a0 = 0;
        if (tb + tid < e1) {
          uint4 e;
          if (paths) {
            e = cl_load4(&L.cand[tb + tid]);
          } else {
            e.x = cl_load(&L.f_xbeg[tb + tid]);
            e.w = cl_load(&L.f_xdeg[tb + tid]);
            e.y = g.off[e.x].y;
            e.z = g.off[e.x + 1].y;
          }
          key = (uint32_t)(cl_load(&cur[e.x]) >> 32);
          if (key <= kcutb && (paths || e.w == lvl)) d = e.z - e.y;
          a0 = e.y;
        }
        uint32_t tot;
        S.pre[tid] = block_excl_scan(d, S.bs, par, &tot);
        S.beg[tid] = a0;
        S.key[tid] = key;
        __syncthreads();
        const uint32_t m = e1 - tb < kClTile ? e1 - tb : kClTile;
        uint32_t round = 0;
        for (uint32_t b = 0; b < tot; b += kThreads) {
          const uint32_t it = b + tid;
          const bool on = it < tot;
          uint32_t dst = 0, xk = kNoArc, arc = 0, xd = 0;
          if (on) {
            const uint32_t j = cl_find(S.pre, m, it);
            const uint32_t a = S.beg[j] + (it - S.pre[j]);
            float x = key_cost(S.key[j]);
            if (paths) {
              const uint4 h = g.phead[2 * (size_t)a], hw = g.phead[2 * (size_t)a + 1];
              const uint32_t k = h.w & 0xffu;
              if (k > 1u) {
                x = canon(x + __uint_as_float(hw.x));
                if (k > 2u) x = canon(x + __uint_as_float(hw.y));
                if (k > 3u) x = canon(x + __uint_as_float(hw.z));
                if (k > 4u) x = canon(x + __uint_as_float(hw.w));
                const float* tw = g.ptail + (size_t)a * g.pstride;
                for (uint32_t i = 4; i + 1 < k; ++i) x = canon(x + tw[i]);
              }
              xk = cost_key(canon(x + __uint_as_float(h.z)));
              dst = h.x;
              arc = h.y;
              xd = h.w >> 8;
            } else {
              const uint4 r = g.xarc[a];
              xk = cost_key(canon(x + __uint_as_float(r.y)));
              dst = r.x;
              arc = r.w;
              xd = r.z;  // the level, or kNoEps
            }
          }
          const bool first = relax(on, dst, xk, arc);
          // (a state reached by a path: only its epsilon arcs count, its own
          // paths are longer paths of the table)
          if (first && (paths ? xd != 0u : xd != kNoEps)) cl_bucket_level(F, L, dst, xd);
          if (++round % kClRounds == 0) cl_flush(S, F, L, paths);
        }
        cl_flush(S, F, L, paths);
      }
      cl_barrier(C, N, gen);
    }
    if (nlev == 0) cl_barrier(C, N, gen);
    if (cl_load(&C->bad)) {
      status = kStatusInternal;
      break;
    }
    stamp(t, 2);
    // ------------------------------------------------------- C: survivors
    const uint32_t nt = cl_load(&F->n_touched);
    if (w == 0 && tid == 0 && nt > S.out.need_frame) S.out.need_frame = nt;
    if (nt > L.frame_cap) {
      status = 4;
      ovf |= kOvfFrame;
      break;
    }
    uint64_t eps = 0;  // epsilon arcs of the closure's states within the cutoff
    {
      uint32_t n = cl_load(&F->n_bk);
      for (uint32_t i = w * kThreads + tid; i < n; i += N * kThreads) {
        const uint4 e = cl_load4(&L.cand[i]);
        if ((uint32_t)(cl_load(&cur[e.x]) >> 32) <= kcutb) eps += e.w;
      }
      n = cl_load(&F->n_bx);
      for (uint32_t i = w * kThreads + tid; i < n; i += N * kThreads) {
        const uint32_t s = cl_load(&L.f_xbeg[i]);
        const uint32_t xd = paths ? cl_load(&L.f_xdeg[i]) : g.off[s + 1].y - g.off[s].y;
        if ((uint32_t)(cl_load(&cur[s]) >> 32) <= kcutb) eps += xd;
      }
    }
    // (the slots are emptied only after every workgroup has counted)
    // the next frame's log-likelihood row on its way to the L2 (no value has
    // this payload)
    if (t < T)
      for (uint32_t k = (w * kThreads + tid) * 32u; k < g.P; k += N * kThreads * 32u)
        my_links += __float_as_uint(L.ll[(size_t)t * g.P + k]) == 0x7fc00001u;
    const bool may_bind = prm.max_active > 0 && nt > (uint32_t)prm.max_active;
    const uint32_t span = kcutb - best_key;
    const uint32_t nbits = span ? 32u - (uint32_t)__clz(span) : 0u;
    uint32_t shift = nbits > 11u ? nbits - 11u : 0u;
    const uint32_t i0 = (uint32_t)((uint64_t)nt * w / N), i1 = (uint32_t)((uint64_t)nt * (w + 1) / N);
    uint32_t my_ns = 0;  // survivors of this workgroup's share, in its part of the survivor arrays
    if (tid == 0) S.base = 0;
    __syncthreads();
    // (the first kHeld states of each thread stay in registers until the
    // frame's end)
    uint32_t hs[kHeld], hk[kHeld];
#pragma unroll
    for (uint32_t u = 0; u < kHeld; ++u) {
      const uint32_t i = i0 + u * kThreads + tid;
      hs[u] = i < i1 ? cl_load(&L.touched[i]) : 0u;
    }
#pragma unroll
    for (uint32_t u = 0; u < kHeld; ++u) {
      const uint32_t i = i0 + u * kThreads + tid;
      hk[u] = i < i1 ? (uint32_t)(cl_load(&cur[hs[u]]) >> 32) : 0u;
    }
    uint32_t turn = 0;
    for (uint32_t b = i0; b < i1; b += kThreads, ++turn) {
      const uint32_t i = b + tid;
      uint32_t s = 0, key = 0xffffffffu;
      if (turn < kHeld) {
#pragma unroll
        for (uint32_t u = 0; u < kHeld; ++u)
          if (turn == u) {
            s = hs[u];
            key = hk[u];
          }
      } else if (i < i1) {
        s = cl_load(&L.touched[i]);
        key = (uint32_t)(cl_load(&cur[s]) >> 32);
      }
      const bool keep = i < i1 && key <= kcutb;
      if (may_bind) {
        if (keep) (void)atomicAdd(&S.hist[(key - best_key) >> shift], 1u);
        const uint32_t p = wave_append(keep, &S.base);
        if (keep) {
          L.surv_pack[i0 + p] = key;
        }
      } else if (keep) {
        cl_mark(C, L, sum, t, wsh, s);
      }
    }
    __syncthreads();
    my_ns = S.base;
    eps = block_sum64(eps, S.bs, par);
    if (tid == 0 && eps) cl_add<unsigned long long>(&F->eps, eps);
    if (may_bind) {
      if (tid == 0 && my_ns) cl_add<uint32_t>(&F->n_surv, my_ns);
      cl_merge_hist(S, C->hist[0]);
    }
    // (late helpers: a launch's workgroups come up over tens of microseconds)
    if (w == 0 && tid == 0 && N < kClMax) {
      const uint32_t here = cl_load(&C->alive) + 1u;
      if (here > N && frames >= kRegroupFrames) cl_store(&F->regroup, 1u);
    }
    cl_barrier(C, N, gen);
    stamp(t, 3);
    regroup = cl_load(&F->regroup) != 0;
    ++frames;
    if (w == 0 && tid == 0) S.out.eps += cl_load(&F->eps);
    cut_key = kcutb;
    // ---------------------------------------- D, E: max-active, kept tokens
    if (may_bind) {
      const uint32_t ns = cl_load(&F->n_surv);
      if (ns > (uint32_t)prm.max_active) {
        uint32_t rank = (uint32_t)prm.max_active, prefix = 0, bits = nbits - shift;
        for (uint32_t d = 0;; ++d) {
          uint32_t bin, before, cnt;
          cl_select_bin(C->hist[d], rank, S, par, &bin, &before, &cnt);
          prefix = (prefix << bits) | bin;
          rank -= before;
          if (shift == 0) break;
          const uint32_t nsh = shift > 11u ? shift - 11u : 0u;
          bits = shift - nsh;
          for (uint32_t i = tid; i < my_ns; i += kThreads) {
            const uint32_t k = (uint32_t)cl_load(&L.surv_pack[i0 + i]) - best_key;
            if ((k >> shift) == prefix) (void)atomicAdd(&S.hist[(k >> nsh) & ((1u << bits) - 1u)], 1u);
          }
          shift = nsh;
          cl_merge_hist(S, C->hist[d + 1]);
          cl_barrier(C, N, gen);
        }
        const uint32_t vkey = best_key + prefix;
        cut_key = vkey < kcutb ? vkey : kcutb;
      }
      stamp(t, 4);
    }
    // the frame's emitting links: candidates within the cutoff
    if (my_work <= kClCand) {
      for (uint32_t i = tid; i < my_work; i += kThreads) my_links += S.cand[i] <= cut_key && S.cand[i] < kInfKey;
    } else {
      // more than LDS holds: formed again from the tokens
      for (uint32_t tb = n0; tb < n1; tb += kClTile) {
        const uint32_t m = n1 - tb < kClTile ? n1 - tb : kClTile;
        uint32_t deg = 0;
        if (tid < m) {
          const uint32_t p = tb + tid;
          const uint32_t s = cl_load(&L.f_state[p]), a0 = g.off[s].x;
          deg = g.off[s + 1].x - a0;
          S.beg[tid] = a0;
          S.key[tid] = cl_load(&L.f_key[p]);
        }
        uint32_t tot;
        S.pre[tid] = block_excl_scan(deg, S.bs, par, &tot);
        __syncthreads();
        for (uint32_t it = tid; it < tot; it += kThreads) {
          const uint32_t j = cl_find(S.pre, m, it);
          const uint4 r = g.earc[S.beg[j] + (it - S.pre[j])];
          float x = key_cost(S.key[j]) + -row[(r.z & 0xffffffu) - 1u];
          x = canon(x + __uint_as_float(r.y));
          const uint32_t xk = cost_key(x);
          my_links += xk <= cut_key && xk < kInfKey;
        }
        __syncthreads();
      }
    }
    // emptied slots: states touched but not kept
    auto finish = [&](uint32_t s, uint32_t key) {
      if (key > cut_key) cur[s] = kEmpty;
      else if (may_bind) cl_mark(C, L, sum, t, wsh, s);
    };
#pragma unroll
    for (uint32_t u = 0; u < kHeld; ++u)
      if (i0 + u * kThreads + tid < i1) finish(hs[u], hk[u]);
    for (uint32_t i = i0 + kHeld * kThreads + tid; i < i1; i += kThreads) {
      const uint32_t s = cl_load(&L.touched[i]);
      finish(s, (uint32_t)(cl_load(&cur[s]) >> 32));
    }
    if (may_bind) {
      cl_barrier(C, N, gen);
    } else {
      stamp(t, 4);
    }
    stamp(t, 5);
    small = nt <= kSmallTouched;
    ++t;
  }

  // ------------------------------------------------------- end of the run
  // (uniform over the cluster: every exit above follows from shared values)
  my_links = block_sum64(my_links, S.bs, par);
  if (tid == 0 && my_links) cl_add<unsigned long long>(&C->links, my_links);
  if (status == 0) cl_barrier(C, N, gen);
  if (w != 0) return;
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
  // the frontier as the LDS path resumes from it: arc ranges, degree prefix sums
  uint32_t W = 0;
  if (status == 0 && (t <= T || L.open)) {
    for (uint32_t b = 0; b < n_all; b += kThreads) {
      const uint32_t p = b + tid;
      uint32_t d = 0;
      if (p < n_all) {
        const uint32_t s = cl_load(&L.f_state[p]);
        const uint32_t a0 = g.off[s].x;
        d = g.off[s + 1].x - a0;
        L.f_ebeg[p] = a0;
      }
      uint32_t tot;
      const uint32_t ex = W + block_excl_scan(d, S.bs, par, &tot);
      W += tot;
      if (p < n_all) L.f_edeg[p] = ex;
    }
    if (tid == 0) L.f_edeg[n_all] = W;
  }
  cl_drain();
  __syncthreads();
  if (tid == 0) {
    S.out.t = t;
    S.out.status = status;
    S.out.ovf = ovf;
    S.out.n_prev = n_all;
    S.out.W = W;
    S.out.hist_ok = hist_ok ? 1u : 0u;
    S.out.node_base = nb;
    S.out.links = cl_load(&C->links);
    S.out.again = regroup && !(small && n_all <= kSmallTokens) ? 1u : 0u;
  }
  __syncthreads();
}

// ------------------------------------------------------------ runs, helpers

// The lane of a helper workgroup (blockIdx.x >= B): helpers go to the XCDs in
// turn, as the leaders do, so it is one whose leader is expected on this
// workgroup's XCD; false: there is none.
__device__ __forceinline__ bool helper_lane(uint32_t B, uint32_t* lane) {
  const uint32_t x = blockIdx.x % kXcds, nl = B > x ? (B - x + kXcds - 1) / kXcds : 0u;
  if (nl == 0) return false;
  *lane = x + kXcds * (((blockIdx.x - B) / kXcds) % nl);
  return true;
}

// The leader opens run number `run` at frame t with whatever helpers answer;
// returns the number of workgroups.  Whole workgroup (`go`: a word of its
// LDS); the frontier of frame t - 1 is in the workspace.
__device__ __forceinline__ uint32_t cl_open(Ctl* C, uint32_t& go, int t, uint32_t n_prev, uint64_t node_base,
                                            bool hist_ok, bool clear, uint32_t run) {
  cl_drain();
  __syncthreads();
  if (threadIdx.x < 64u) {
    if (threadIdx.x == 0) {
      cl_store(&C->t, (uint32_t)t);
      cl_store(&C->n_prev, n_prev);
      cl_store(&C->node_base, (uint32_t)node_base);
      cl_store(&C->node_base_hi, (uint32_t)(node_base >> 32));
      cl_store(&C->hist_ok, hist_ok ? 1u : 0u);
      cl_store(&C->clear, clear ? 1u : 0u);
      cl_store(&C->bar0, cl_load(&C->bar));
      cl_drain();
      cl_store(&C->cmd, run);
    }
    // the helpers that have answered when the wait ends are in the run
    const uint64_t t0 = wall_clock64();
    uint64_t mask;
    do {
      mask = __ballot(threadIdx.x < kClMax && cl_load(&C->join[threadIdx.x % kClMax]) == run);
    } while ((uint32_t)__popcll(mask) < cl_load(&C->alive) && wall_clock64() - t0 < kJoinTicks);
    if (threadIdx.x == 0) {
      cl_store<unsigned long long>(&C->members, ((unsigned long long)run << 32) | mask);
      go = (uint32_t)__popcll(mask) + 1u;
    }
  }
  __syncthreads();
  const uint32_t N = go;
  __syncthreads();
  return N;
}

// A helper (its number in id, kClMax before it has one) waits for the leader's
// next run: its place and the number of
// workgroups as place << 8 | number, or 0 when it leaves (the leader is done,
// is on another XCD, has enough helpers, or opens no run for idle_ticks).
// Whole workgroup.
__device__ __forceinline__ uint32_t cl_wait(Ctl* C, uint32_t& go_lds, uint32_t& seen, uint32_t& id,
                                            uint64_t idle_ticks) {
  __syncthreads();
  if (threadIdx.x == 0) {
    const uint64_t idle = wall_clock64();
    uint32_t go = 0;
    while (true) {
      if (cl_load(&C->quit) || wall_clock64() - idle > idle_ticks) break;
      if (id == kClMax) {
        const uint32_t x = cl_load(&C->xcc);
        if (x == 0) {
          __builtin_amdgcn_s_sleep(16);
          continue;
        }
        if (x - 1u != cl_xcc()) break;
        const uint32_t ticket = cl_add<uint32_t>(&C->tickets, 1u);
        if (ticket >= kClMax - 1u) break;
        id = ticket;
        cl_add<uint32_t>(&C->alive, 1u);
      }
      const uint32_t run = cl_load(&C->cmd);
      if (run == seen) {
        __builtin_amdgcn_s_sleep(8);
        continue;
      }
      // answer, and see whether the leader took it in
      seen = run;
      cl_store(&C->join[id], run);
      SpinClock spin(wall_clock64());
      unsigned long long m = cl_load(&C->members);
      while ((uint32_t)(m >> 32) != run && cl_load(&C->cmd) == run && !spin.beyond(wall_clock64()))
        m = cl_load(&C->members);
      if ((uint32_t)(m >> 32) != run || !((m >> id) & 1u)) continue;
      const uint32_t mask = (uint32_t)m;
      go = (((uint32_t)__popc(mask & ((1u << id) - 1u)) + 1u) << 8) | ((uint32_t)__popc(mask) + 1u);
      break;
    }
    if (go == 0 && id < kClMax) (void)cl_add<uint32_t>(&C->alive, ~0u);
    go_lds = go;
  }
  __syncthreads();
  const uint32_t go = go_lds;
  __syncthreads();
  return go;
}

}  // namespace wd
