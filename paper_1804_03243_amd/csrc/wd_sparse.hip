// Lattice pruning of large frames without a raw lattice (Sec. 3.5), from the
// node store, the graph's in-arcs and the log-likelihoods.
//
// A frame of thousands of tokens and more has as many raw links, of which the
// lattice beam keeps a handful (hundreds, of a million, on wide beams).  A
// link's extra cost is its destination's plus a difference that is not
// negative, so a link is kept only if its destination's extra cost is within
// the lattice beam, and only such "live" nodes' extra costs decide anything.
// The backward sweep therefore starts from the last frame's live nodes and
// walks live nodes' in-arcs only: for each, the token of the arc's source
// state (found among its frame's nodes, sorted by state), the link's cost by
// the forward pass's own additions, the frame's cutoff (whether the link
// exists), and an atomic minimum into the source's extra cost.  Extra costs
// only fall, so a node whose extra cost falls again within its frame (through
// epsilon links) is simply walked again until nothing changes: the fixpoint of
// the paper's recursion, the same values bit for bit.  The kept links are then
// formed frame by frame, all frames at once, in the layout the lattice pass
// reads, out of the live nodes in state order.
//
// The sweep is a latency chain over the frames (node, in-arc offsets, in-arcs,
// source lookup, its token, minimum), so a cluster of workgroups on one XCD
// runs it (wd_cluster.h), each with the states of three frames in LDS: all of
// them, or every 2^k-th when a frame has more than kSpWin.
//
// A generation's nodes are shared out whole, so the in-arcs of a state that many
// arcs end in (the back-off states of a language model have 10^5 and more) would
// fall to one workgroup, and may be far more than the arcs out of the frame's
// tokens, which alone can be links.  Such hubs are left to a second step, all
// workgroups together: over shares of their in-arcs, or, where these are more,
// over the tokens' out-arcs into them.
#include "wd_cluster.h"
#include "wd_host.h"
#include "wd_sparse.h"

namespace wd {

constexpr uint32_t kSpTok = kThreads;          // live nodes per tile
constexpr uint32_t kSpWin = 8192;              // states of one frame held in LDS
constexpr uint32_t kSpPer = kSpWin / kThreads;  // loaded per thread
constexpr uint64_t kSpGather = 300;            // helpers have 3 µs to come up,
constexpr uint64_t kSpGatherWide = 10000;      // 100 µs where frames average more than
constexpr uint64_t kSpWide = 30000;            // this many tokens
constexpr uint32_t kSpHelpers = 28;            // (an XCD's CUs, but for a few)
// A node is a hub from kSpHubMin in-arcs on where there are as many nodes as the
// frame's tokens, and from kSpHubMax on in any case (two rounds of a workgroup; the
// second step costs a barrier and a tile, about 5 µs).  Between the two the nodes'
// in-arcs together stay within the tokens' out-arcs, taken as kSpOut per token
// (with its own offsets to read).
constexpr uint32_t kSpHubMin = 32, kSpHubMax = 2048, kSpOut = 3;
constexpr uint32_t kSpHubs = 4096;             // hubs listed; more are left to the out-arcs

struct SpShared {
  BlockScratch bs;
  uint32_t win[3][kSpWin];
  uint32_t pre[kSpTok], beg[kSpTok], key[kSpTok], arc[kSpTok], ex[kSpTok], node[kSpTok];
  uint32_t go;
};

// Counters of a sweep, in the histograms of the control block.
struct SpCounters {
  WD_GLOBAL uint32_t* x;    // [3] work-list entries pushed by a generation
  WD_GLOBAL uint32_t* e;    // [3] nodes of the frame before, pushed by a frame
  WD_GLOBAL uint32_t* any;  // a final state was reached
  WD_GLOBAL unsigned long long* best;  // inverted (final cost key, node offset) of the best end token
  WD_GLOBAL uint32_t* h;    // [3] hubs among a generation's nodes
  WD_GLOBAL unsigned long long* ha;  // [3] their in-arcs
  WD_GLOBAL uint32_t* hubs;  // [kSpHubs] of this generation
};
__device__ __forceinline__ SpCounters sp_counters(const LaneDesc& L) {
  WD_GLOBAL uint32_t* h = &((Ctl*)L.ctl)->hist[0][0];
  return SpCounters{h, h + 32, h + 64, (WD_GLOBAL unsigned long long*)(h + 96),
                    h + 128, (WD_GLOBAL unsigned long long*)(h + 160), h + 256};
}
constexpr uint32_t kSpCounterWords = 192;
static_assert(256 + kSpHubs <= kClDigits * kHistBins, "the hubs' list behind the counters");

// Appends v to list[] for every lane with `on`: one add per wavefront.  Whole
// wavefronts.  Entries beyond the capacity are dropped; the count tells.
__device__ __forceinline__ void sp_push(bool on, uint32_t v, WD_GLOBAL uint32_t* list, uint64_t cap,
                                        WD_GLOBAL uint32_t* n) {
  const uint64_t m = __ballot(on);
  if (!m) return;
  const int first = __ffsll((unsigned long long)m) - 1;
  uint32_t base = 0;
  if ((int)lane_id() == first) base = cl_add<uint32_t>(n, (uint32_t)__popcll(m));
  base = (uint32_t)__builtin_amdgcn_readlane((int)base, first);
  const uint32_t p = base + rank_in(m);
  if (on && p < cap) cl_store(&list[p], v);
}

// Chip-wide mode, before the sweep: every node's extra cost is +inf, the
// control block is clean.  (In one-workgroup mode the sweep and the kernels
// before the forward pass do this.)
__global__ void __launch_bounds__(256) k_sp_init(const LaneDesc* __restrict__ lanes, uint32_t flags) {
  const LaneDesc& L = lanes[blockIdx.y];
  if (!sparse_lane(L, flags)) return;
  const uint64_t n = L.node_off[L.T + 1];
  for (uint64_t i = (uint64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (uint64_t)gridDim.x * 256)
    L.extra_key[i] = kInfKey;
  if (blockIdx.x == 0)
    for (uint32_t i = threadIdx.x; i < kCtlHead / 4u; i += 256)
      ((WD_GLOBAL uint32_t*)L.ctl)[sizeof(ClusterCtl) / 4u + i] = 0;
}

// The sweep, workgroup w of N.
__device__ __forceinline__ void sp_sweep(const DevGraph& g, const LaneDesc& L, SpShared& S, Ctl* C, uint32_t w,
                                         uint32_t N, uint32_t lb_key, bool fill) {
  const uint32_t tid = threadIdx.x;
  const int T = L.T;
  const SpCounters cn = sp_counters(L);
  uint32_t par = 0, gen = cl_load(&C->bar0);
  const uint64_t cap = L.node_cap;
  if (fill) {
    const uint64_t n = L.node_off[T + 1], lo = n * w / N, hi = n * (w + 1) / N;
    for (uint64_t i = lo + tid; i < hi; i += kThreads) cl_store(&L.extra_key[i], kInfKey);
  }
  if (w == 0 && tid < kSpCounterWords) cl_store(&cn.x[tid], 0u);
  cl_barrier(C, N, gen);
  WD_GLOBAL uint32_t* const we = (WD_GLOBAL uint32_t*)L.alpha;  // two frames' lists (node_cap entries each)
  WD_GLOBAL uint32_t* const wx = (WD_GLOBAL uint32_t*)L.beta;   // two generations' lists
  // ------------------------------------------------ final costs, best end token
  const uint64_t nT0 = L.node_off[T], nT1 = L.node_off[T + 1];
  bool final_used = false;
  if (g.final_w) {
    uint32_t any = 0;
    for (uint64_t n = nT0 + w * kThreads + tid; n < nT1; n += N * kThreads) {
      const float fw = g.final_w[L.n_state[n]];
      const float c = key_cost((uint32_t)(L.n_pack[n] >> 32));
      any |= (fw < INFINITY && (c + fw) < INFINITY) ? 1u : 0u;
    }
    any = block_or(any, S.bs, par);
    if (tid == 0 && any) cl_add<uint32_t>(cn.any, 1u);
    cl_barrier(C, N, gen);
    final_used = cl_load(cn.any) != 0;
  }
  auto final_cost = [&](uint64_t n) -> float {
    const float c = key_cost((uint32_t)(L.n_pack[n] >> 32));
    return final_used ? canon(c + g.final_w[L.n_state[n]]) : c;
  };
  uint64_t m = kEmpty;
  for (uint64_t n = nT0 + w * kThreads + tid; n < nT1; n += N * kThreads) {
    const uint64_t v = pack_tok(cost_key(final_cost(n)), (uint32_t)(n - nT0));
    m = v < m ? v : m;
  }
  m = block_min64(m, S.bs, par);
  if (tid == 0)
    (void)__hip_atomic_fetch_max(cn.best, ~(unsigned long long)m, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  cl_barrier(C, N, gen);
  m = ~cl_load(cn.best);
  const uint32_t best_key = (uint32_t)(m >> 32);
  if (w == 0 && tid == 0) {
    LaneInfo* I = L.info;
    I->final_used = final_used ? 1 : 0;
    I->best_node = (uint32_t)(nT0 + (m & 0xffffffffu));
    I->best_cost = key_cost(best_key);
  }
  if (best_key >= kInfKey) return;  // (the lattice kernel reports it)
  const float best = key_cost(best_key);
  // the last frame's live nodes
  for (uint64_t b = nT0 + w * kThreads; b < nT1; b += N * kThreads) {
    const uint64_t n = b + tid;
    uint32_t e = kInfKey;
    if (n < nT1) {
      const float F = final_cost(n);
      if (F < INFINITY) e = cost_key(F - best);
      if (e < kInfKey) cl_store(&L.extra_key[n], e);
    }
    const bool live = e <= lb_key;
    if (live) (void)__hip_atomic_fetch_or(&L.used[n >> 5], 1u << (n & 31u), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    sp_push(live, (uint32_t)n, we + (size_t)((T + 1) & 1) * cap, cap, &cn.e[(T + 1) % 3]);
  }
  // the windows of the last two frames
  SpFrame f0 = sp_frame(L, T, kSpWin), f1 = sp_frame(L, T - 1, kSpWin);
  for (uint32_t i = tid; i < f0.m; i += kThreads) S.win[T % 3][i] = L.n_state[f0.n0 + ((uint64_t)i << f0.k)];
  if (T > 0)
    for (uint32_t i = tid; i < f1.m; i += kThreads)
      S.win[(T - 1) % 3][i] = L.n_state[f1.n0 + ((uint64_t)i << f1.k)];
  cl_barrier(C, N, gen);

  uint32_t gi = 0;
  uint32_t n_e = cl_load(&cn.e[(T + 1) % 3]);  // nodes of the next frame to walk, pushed by this one
  for (int t = T; t >= 0; --t) {
    const uint32_t* const win0 = S.win[t % 3];
    const uint32_t* const win1 = S.win[(t + 2) % 3];  // frame t - 1
    // frame t - 2's states, on their way while frame t is walked
    const SpFrame f2 = sp_frame(L, t - 2, kSpWin);
    uint32_t ahead[kSpPer];
#pragma unroll
    for (uint32_t u = 0; u < kSpPer; ++u) {
      const uint32_t i = tid + u * kThreads;
      ahead[u] = i < f2.m ? L.n_state[f2.n0 + ((uint64_t)i << f2.k)] : 0u;
    }
    const uint32_t cut = cost_key(L.cut[t]);
    const float* row = (const float*)L.ll + (size_t)(t > 0 ? t - 1 : 0) * g.P;
    if (w == 0 && tid == 0) cl_store(&cn.e[(t + 2) % 3], 0u);  // (frame t - 1's)
    // A link out of node src, of cost x, into node `node` (cost key, predecessor
    // arc and extra cost given): whether src is to be walked (again) in this
    // frame (epsilon links), in the frame before.
    auto relax = [&](bool eps, uint32_t src, float x, uint32_t arc_id, uint32_t node, uint32_t key, uint32_t arc,
                     uint32_t ex, bool& push_x, bool& push_e) {
      const uint32_t xk = cost_key(x);
      if (xk > cut || xk >= kInfKey) return;
      // the link that made the destination's token names its predecessor
      if (xk == key && arc_id == arc) L.n_pred[node] = src;
      const uint32_t le = cost_key(key_cost(ex) + (x - key_cost(key)));
      if (le > lb_key) return;
      const uint32_t old = __hip_atomic_fetch_min(&L.extra_key[src], le, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      const bool fresh = old > lb_key;
      if (fresh)
        (void)__hip_atomic_fetch_or(&L.used[src >> 5], 1u << (src & 31u), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      push_x = eps && le < old;
      push_e = !eps && fresh;
    };
    auto push = [&](bool push_x, bool push_e, uint32_t src) {
      sp_push(push_x, src, wx + (size_t)(gi & 1) * cap, cap, &cn.x[gi % 3]);
      sp_push(push_e, src, we + (size_t)(t & 1) * cap, cap, &cn.e[t % 3]);
    };
    // In-arcs of nodes i0 .. i1 of a list (`all`: of the frame): all of those
    // with up to `lim`; or (`shared`) this workgroup's part of each node's.
    auto walk = [&](const WD_GLOBAL uint32_t* list, bool all, uint32_t i0, uint32_t i1, uint32_t lim, bool shared) {
      for (uint32_t tb = i0; tb < i1; tb += kSpTok) {
        const uint32_t mm = i1 - tb < kSpTok ? i1 - tb : kSpTok;
        uint32_t deg = 0, beg = 0, key = 0, arc = 0, ex = kInfKey, v = 0;
        bool hub = false;
        if (tid < mm) {
          v = all ? (uint32_t)(f0.n0 + tb + tid) : cl_load(&list[tb + tid]);
          const uint32_t s = L.n_state[v];
          const unsigned long long pk = L.n_pack[v];
          ex = cl_load(&L.extra_key[v]);
          const uint32_t r0 = g.roff[s], r1 = g.roff[s + 1];
          key = (uint32_t)(pk >> 32);
          arc = (uint32_t)pk;
          beg = r0;
          deg = ex <= lb_key ? r1 - r0 : 0u;
          if (shared) {
            const uint32_t d = deg;
            beg += (uint32_t)((uint64_t)d * w / N);
            deg = (uint32_t)((uint64_t)d * (w + 1) / N) - (uint32_t)((uint64_t)d * w / N);
          } else {
            hub = deg > lim;
          }
        }
        if (!shared) {
          if (hub) {
            cl_add<unsigned long long>(&cn.ha[gi % 3], (unsigned long long)deg);
            deg = 0;
          }
          sp_push(hub, v, cn.hubs, kSpHubs, &cn.h[gi % 3]);
        }
        uint32_t tot;
        S.pre[tid] = block_excl_scan(deg, S.bs, par, &tot);
        S.beg[tid] = beg;
        S.key[tid] = key;
        S.arc[tid] = arc;
        S.ex[tid] = ex;
        S.node[tid] = v;
        __syncthreads();
        for (uint32_t b = 0; b < tot; b += kThreads) {
          const uint32_t it = b + tid;
          bool push_x = false, push_e = false;
          uint32_t src = ~0u;
          if (it < tot) {
            const uint32_t j = cl_find(S.pre, mm, it);
            const uint4 r = g.rarc[S.beg[j] + (it - S.pre[j])];  // {source state, weight, ilabel, arc}
            const bool eps = r.z == 0;
            if (eps) src = sp_lookup<kSpWin>(L, f0, win0, r.x);
            else if (t > 0) src = sp_lookup<kSpWin>(L, f1, win1, r.x);
            if (src != ~0u) {
              float x = key_cost((uint32_t)(L.n_pack[src] >> 32));
              if (!eps) x = x + -row[r.z - 1u];
              x = canon(x + __uint_as_float(r.y));
              relax(eps, src, x, r.w, S.node[j], S.key[j], S.arc[j], S.ex[j], push_x, push_e);
            }
          }
          push(push_x, push_e, src);
        }
        __syncthreads();
      }
    };
    // The out-arcs of this workgroup's share of the source frame's tokens into
    // live nodes of more than `lim` in-arcs.
    auto from_tokens = [&](bool eps, uint32_t lim) {
      const SpFrame& f = eps ? f0 : f1;
      const uint32_t i1 = (uint32_t)((uint64_t)f.n * (w + 1) / N);
      for (uint32_t tb = (uint32_t)((uint64_t)f.n * w / N); tb < i1; tb += kSpTok) {
        const uint32_t mm = i1 - tb < kSpTok ? i1 - tb : kSpTok;
        uint32_t deg = 0, beg = 0, key = 0;
        const uint32_t v = (uint32_t)(f.n0 + tb + tid);
        if (tid < mm) {
          const uint32_t s = L.n_state[v];
          const uint4 o0 = g.off[s], o1 = g.off[s + 1];
          key = (uint32_t)(L.n_pack[v] >> 32);
          beg = eps ? o0.y : o0.x;
          deg = eps ? o1.y - o0.y : o1.x - o0.x;
        }
        uint32_t tot;
        S.pre[tid] = block_excl_scan(deg, S.bs, par, &tot);
        S.beg[tid] = beg;
        S.key[tid] = key;
        S.node[tid] = v;
        __syncthreads();
        for (uint64_t b = 0; b < tot; b += kThreads) {
          const uint64_t it = b + tid;
          bool push_x = false, push_e = false;
          uint32_t src = ~0u;
          if (it < tot) {
            const uint32_t j = cl_find(S.pre, mm, (uint32_t)it);
            const uint32_t a = S.beg[j] + ((uint32_t)it - S.pre[j]);
            const uint4 r = eps ? g.xarc[a] : g.earc[a];  // {destination, weight, ilabel | level, arc}
            const uint32_t dn = g.roff[r.x + 1] - g.roff[r.x] > lim ? sp_lookup<kSpWin>(L, f0, win0, r.x) : ~0u;
            if (dn != ~0u) {
              const uint32_t ex = cl_load(&L.extra_key[dn]);
              if (ex <= lb_key) {
                src = S.node[j];
                float x = key_cost(S.key[j]);
                if (!eps) x = x + -row[(r.z & 0xffffffu) - 1u];
                x = canon(x + __uint_as_float(r.y));
                const unsigned long long pk = L.n_pack[dn];
                relax(eps, src, x, r.w, dn, (uint32_t)(pk >> 32), (uint32_t)pk, ex, push_x, push_e);
              }
            }
          }
          push(push_x, push_e, src);
        }
        __syncthreads();
      }
    };
    bool first = true;
    uint32_t n_list = n_e;
    while (true) {
      // this generation's nodes: the frame's list, or what the last
      // generation pushed (all live nodes of the frame, if that overflowed)
      const WD_GLOBAL uint32_t* list = first ? we + (size_t)((t + 1) & 1) * cap : wx + (size_t)((gi + 1) & 1) * cap;
      const bool all = n_list > cap;
      if (all) n_list = f0.n;
      if (w == 0 && tid == 0) {
        cl_store(&cn.x[(gi + 1) % 3], 0u);
        cl_store(&cn.h[(gi + 1) % 3], 0u);
        cl_store<unsigned long long>(&cn.ha[(gi + 1) % 3], 0ull);
      }
      const uint64_t out = (uint64_t)kSpOut * ((uint64_t)f0.n + f1.n);
      uint32_t lim = kSpHubMax;
      if (out / kSpHubMax < n_list) {
        lim = (uint32_t)((float)out / (float)n_list);
        lim = lim > kSpHubMin ? lim : kSpHubMin;
      }
      walk(list, all, (uint32_t)((uint64_t)n_list * w / N), (uint32_t)((uint64_t)n_list * (w + 1) / N), lim, false);
      cl_barrier(C, N, gen);
      // (every word the next steps depend on in one round of loads)
      const uint32_t n_hub = cl_load(&cn.h[gi % 3]);
      uint32_t bad = cl_load(&C->bad), n_x = cl_load(&cn.x[gi % 3]);
      n_e = cl_load(&cn.e[t % 3]);
      if (bad) return;
      if (n_hub) {
        if (n_hub <= kSpHubs && cl_load(&cn.ha[gi % 3]) <= out) {
          walk(cn.hubs, false, 0, n_hub, 0, true);
        } else {
          if (t > 0) from_tokens(false, lim);
          from_tokens(true, lim);
        }
        cl_barrier(C, N, gen);
        bad = cl_load(&C->bad);
        n_x = cl_load(&cn.x[gi % 3]);
        n_e = cl_load(&cn.e[t % 3]);
        if (bad) return;
      }
      first = false;
      ++gi;
      if (n_x == 0) break;
      n_list = n_x;
    }
    // frame t - 2 takes the place of frame t + 1 (whose window nobody reads
    // any more)
#pragma unroll
    for (uint32_t u = 0; u < kSpPer; ++u) {
      const uint32_t i = tid + u * kThreads;
      if (i < f2.m) S.win[(t + 1) % 3][i] = ahead[u];
    }
    f0 = f1;
    f1 = f2;
    __syncthreads();
  }
}

__global__ void __launch_bounds__(kThreads) k_sp_sweep(DevGraph g, const LaneDesc* __restrict__ lanes, Params prm,
                                                       uint32_t B) {
  __shared__ SpShared S;
  const bool lead = blockIdx.x < B;
  uint32_t lane_no = blockIdx.x;
  if (!lead && !helper_lane(B, &lane_no)) return;
  const LaneDesc& L = lanes[lane_no];
  // (one thread looks for all: a helper may come up as late as the leader's last
  // store, which can be to the status)
  if (threadIdx.x == 0) S.go = sparse_lane(L, prm.flags) ? 1u : 0u;
  __syncthreads();
  const bool wanted = S.go != 0;
  __syncthreads();
  if (!wanted) return;
  Ctl* const C = (Ctl*)((WD_GLOBAL char*)L.ctl + sizeof(ClusterCtl));  // (its header only)
  uint32_t w = 0, N = 1;
  if (lead) {
    if (threadIdx.x == 0) cl_store(&C->xcc, cl_xcc() + 1u);
    // Helpers of this launch come up over tens of microseconds; those that have
    // not arrived when the run opens stay out of it.  Frames of a few live
    // nodes gain little from them (and each adds to the barriers); wide ones,
    // with thousands, are worth the wait.
    const bool wide = L.info->tokens > kSpWide * ((uint64_t)L.T + 1);
    const uint64_t t0 = wall_clock64(), limit = wide ? kSpGatherWide : kSpGather;
    if (gridDim.x > B && threadIdx.x == 0)
      while (wall_clock64() - t0 < limit && cl_load(&C->alive) < kSpHelpers) __builtin_amdgcn_s_sleep(2);
    __syncthreads();
    N = cl_open(C, S.go, 0, 0, 0, false, false, 1u);
  } else {
    uint32_t seen = 0;
    uint32_t id = kClMax;
    const uint32_t go = cl_wait(C, S.go, seen, id, kIdleTicks);
    if (go == 0) return;
    w = go >> 8;
    N = go & 0xffu;
  }
  // (an infinite lattice beam keeps every finite extra cost)
  const uint32_t lb = cost_key(prm.lattice_beam);
  sp_sweep(g, L, S, C, w, N, lb < kInfKey ? lb : kInfKey - 1u, (prm.flags & kFlagSwept) == 0);
  if (lead && threadIdx.x == 0) {
    if (cl_load(&C->bad)) L.info->status = kStatusInternal;
    cl_store(&C->quit, 1u);
  }
}

void launch_sweep(const DevGraph& g, const LaneDesc* lanes, int B, const Params& prm, hipStream_t s) {
  if (prm.flags & kFlagSwept) hipLaunchKernelGGL(k_sp_init, dim3(1024, B), dim3(256), 0, s, lanes, prm.flags);
  hipLaunchKernelGGL(k_sp_sweep, dim3(cluster_grid(B)), dim3(kThreads), 0, s, g, lanes, prm, (uint32_t)B);
}

}  // namespace wd
