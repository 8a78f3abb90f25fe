// Lattice links of the one-workgroup decode (Sec. 3.4), written after the
// forward pass from what it recorded, every frame at once.
//
// A link is a token-passing operation whose result is within the frame's
// final cutoff: an emitting arc out of a token of frame t-1 into frame t, or
// an epsilon arc out of a token of frame t.  Its cost is the same fp32 sum
// the forward pass formed (token cost, then the acoustic cost, then the arc
// weight, each addition rounded), so it can be formed again from the node
// store (each frame's tokens in state order, with their cost keys), the
// graph and the log-likelihoods; the forward pass keeps only the per-frame
// node records and cutoffs.  The links of frame t are its emitting links in
// work-item order (frontier of frame t-1 in state order, each token's arcs
// in arc order: arc-id order) followed by its epsilon links (frontier of
// frame t in state order, each token's epsilon arcs in order), exactly the
// layout the lattice pass reads.  Three launches: per-frame counts, one
// workgroup per utterance turning them into offsets (and checking the link
// store's capacity), then the links, each frame by one workgroup (of a small
// frame from the records that the count has kept).
#include "wd_block.h"
#include "wd_host.h"
#include "wd_sparse.h"

namespace wd {

constexpr int kLT = 256;              // threads per workgroup
constexpr int kLWv = kLT / 64;        // wavefronts
constexpr uint32_t kLinkBlocks = 256;  // workgroups per utterance (frames in turn)
constexpr uint32_t kSliceBlocks = 1024;  // chip-wide: workgroups per utterance (slices in turn)
constexpr uint32_t kSpBWin = 2048;     // sparse utterances: states of one frame held in LDS
constexpr uint32_t kSpList = 2048;     // live nodes listed together

// Links of a frame that the count keeps for the write: a frame of a hundred
// tokens has about as many, and 8 KB of LDS leave the count its workgroups per CU.
// Both passes are bound by gathers of arcs and log-likelihoods; with the records
// only the count does them (one utterance of 1000 frames on 5M states: lattice
// stage 1.53 ms before, 1.50 ms with them).
constexpr uint32_t kFound = 512;

struct LinkShared {
  BlockScratch bs;
  uint32_t pre[kLT];    // exclusive prefix of the tile's tokens' arc counts
  uint32_t beg[kLT];    // first arc of each token of the tile
  float cost[kLT];      // token cost
  uint32_t cls[kLT];    // token state's epsilon level (epsilon runs)
  uint4 found[kFound];  // a frame's links, as the count finds them
  unsigned long long base;
};

// The node of state s among one frame's nodes [n0, n1) (sorted by state), or
// ~0 when s has none.
__device__ __forceinline__ uint64_t node_of(const LaneDesc& L, uint64_t n0, uint64_t n1, uint32_t s) {
  uint64_t lo = n0, hi = n1;
  while (lo < hi) {
    const uint64_t mid = (lo + hi) >> 1;
    if (L.n_state[mid] < s) lo = mid + 1;
    else hi = mid;
  }
  return lo < n1 && L.n_state[lo] == s ? lo : ~0ull;
}

// One run of frame t: the emitting links (kEps false; sources: the nodes of
// frame t-1) or the epsilon links (sources: the nodes of frame t).  Counts
// them (kWrite false: returns the count in every thread) or writes them from
// link `at` on (returns the count, sets *xmask and *bad).
// `found` (count mode, or null): the links' records {arc, source node,
// destination state, x bits} go to LDS, up to kFound of them.
template <bool kEps, bool kWrite>
__device__ __forceinline__ uint32_t link_run(const DevGraph& g, const LaneDesc& L, LinkShared& sh, uint32_t& par,
                                             int t, uint32_t cut, uint64_t at, uint32_t* xmask, uint32_t* bad,
                                             bool found = false) {
  const uint32_t tid = threadIdx.x;
  const uint64_t p0 = L.node_off[kEps ? t : t - 1], p1 = L.node_off[kEps ? t + 1 : t];
  const uint64_t d0 = L.node_off[t], d1 = L.node_off[t + 1];  // destinations: frame t
  const float* row = L.ll + (size_t)(t > 0 ? t - 1 : 0) * g.P;
  uint32_t n = 0;  // links of the run so far (write mode: in every thread)
  uint32_t cnt = 0;  // count mode: this thread's links
  for (uint64_t q0 = p0; q0 < p1; q0 += kLT) {
    const uint32_t m = (uint32_t)(p1 - q0 < (uint64_t)kLT ? p1 - q0 : (uint64_t)kLT);
    uint32_t deg = 0, a0 = 0, c = 0;
    float cost = 0.0f;
    if (tid < m) {
      const uint32_t s = L.n_state[q0 + tid];
      cost = key_cost((uint32_t)(L.n_pack[q0 + tid] >> 32));
      const uint4 o0 = g.off[s], o1 = g.off[s + 1];
      a0 = kEps ? o0.y : o0.x;
      deg = kEps ? o1.y - o0.y : o1.x - o0.x;
      if (kEps) c = g.sclass[s];
    }
    uint32_t tot;
    const uint32_t ex = block_excl_scan<kLWv>(deg, sh.bs, par, &tot);
    sh.pre[tid] = ex;
    sh.beg[tid] = a0;
    sh.cost[tid] = cost;
    sh.cls[tid] = c;
    __syncthreads();
    for (uint32_t w0 = 0; w0 < tot; w0 += kLT) {
      const uint32_t w = w0 + tid;
      bool in = false;
      uint32_t j = 0, xb = 0;
      uint4 r = make_uint4(0, 0, 0, 0);
      if (w < tot) {
        j = search_le(sh.pre, m, w);
        const uint32_t a = sh.beg[j] + (w - sh.pre[j]);
        float x;
        if (kEps) {
          r = g.xarc[a];
          x = canon(sh.cost[j] + __uint_as_float(r.y));
        } else {
          r = g.earc[a];
          const float ac = -row[(r.z & 0xffffffu) - 1u];
          x = sh.cost[j] + ac;
          x = canon(x + __uint_as_float(r.y));
        }
        xb = __float_as_uint(x);
        const uint32_t xk = cost_key(x);
        in = xk <= cut && xk < kInfKey;
      }
      if (!kWrite && !found) {
        cnt += in ? 1u : 0u;
        continue;
      }
      uint32_t nsub;
      const uint32_t pos = n + block_excl_scan<kLWv>(in ? 1u : 0u, sh.bs, par, &nsub);
      n += nsub;
      if (!in) continue;
      if (!kWrite) {
        const uint32_t q = (uint32_t)at + pos;
        if (q < kFound) sh.found[q] = make_uint4(r.w, (uint32_t)(q0 + j), r.x, xb);
        continue;
      }
      const uint64_t dn = node_of(L, d0, d1, r.x);
      if (dn == ~0ull) {
        *bad = 1;
        continue;
      }
      const uint32_t src = (uint32_t)(q0 + j);
      L.links[at + pos] = make_uint4(r.w, src, (uint32_t)dn, xb);
      if (kEps) {
        const uint32_t cls = sh.cls[j];
        L.link_lvl[at + pos] = (uint8_t)cls;
        *xmask |= 1u << (cls < 31u ? cls : 31u);
      }
      // the link that made the destination's token names its predecessor
      if (L.n_pack[dn] == pack_tok(cost_key(__uint_as_float(xb)), r.w)) L.n_pred[dn] = src;
    }
    __syncthreads();  // every read of the tile's arrays done before the next tile
  }
  if (!kWrite && !found) {
    uint32_t all;
    (void)block_excl_scan<kLWv>(cnt, sh.bs, par, &all);
    return all;
  }
  return n;
}

// ------------------------------------------------- sparse utterances' links

struct SpLinkShared {
  BlockScratch bs;
  uint32_t win[kSpBWin];
  uint32_t list[kSpList];  // live nodes of a tile, as offsets from its first node
  uint32_t pre[kLT], beg[kLT], node[kLT];
  float cost[kLT];
  uint32_t cls[kLT];
};

// Slices of an utterance's frames: a frame's links are formed by this many
// workgroups, each out of an equal part of the source frame's nodes.  With one
// workgroup a frame, the last frames of a wide decode (every token of the very
// last one within the beam ends a path) took as long as all the others: of 60
// frames of up to 650 thousand tokens, 604 thousand links kept, 9.8 ms each
// for count and write.  A slice costs some 10 µs however few live nodes it has,
// so frames of the one-workgroup mode are one slice.
constexpr uint32_t kSliceNodes = 8192;
__device__ __forceinline__ uint32_t slices_of(const LaneDesc& L, uint32_t flags) {
  if (!(flags & kFlagSwept)) return 1u;
  const uint64_t n = L.info->max_tokens / kSliceNodes;
  return n < 1 ? 1u : n < kSlices ? (uint32_t)n : kSlices;
}

// The kept emitting links into frame t out of frame t - 1's live nodes (kEps
// false), or the kept epsilon links of frame t, those of slice k of ns: counted,
// or written from link `at` on, in the order of their sources' states and arcs.
template <bool kEps, bool kWrite>
__device__ __forceinline__ uint32_t sp_run(const DevGraph& g, const LaneDesc& L, SpLinkShared& sh, uint32_t& par, int t,
                                           uint32_t k, uint32_t ns, const SpFrame& df, uint32_t lb_key, uint64_t at,
                                           uint32_t* xmask) {
  const uint32_t tid = threadIdx.x;
  uint64_t p0 = L.node_off[kEps ? t : t - 1], p1 = L.node_off[kEps ? t + 1 : t];
  if (ns > 1) {  // (cut at words of the live nodes' bitmap)
    const uint64_t w0 = p0 >> 5, n = ((p1 + 31) >> 5) - w0, a = 32 * (w0 + n * k / ns), b = 32 * (w0 + n * (k + 1) / ns);
    if (a > p0) p0 = a;
    if (b < p1) p1 = b;
  }
  const float* row = (const float*)L.ll + (size_t)(t > 0 ? t - 1 : 0) * g.P;
  const uint32_t cut = cost_key(L.cut[t]);
  uint32_t n = 0;
  for (uint64_t q0 = p0 & ~31ull; q0 < p1; q0 += 32u * kLT) {
    // live nodes of a tile, a bitmap word per thread, listed kSpList at a time
    uint32_t word = 0;
    const uint64_t wb = q0 + 32u * tid;
    if (wb < p1) {
      word = L.used[wb >> 5];
      if (wb < p0) word &= ~0u << (p0 - wb);
      if (p1 - wb < 32u) word &= (1u << (p1 - wb)) - 1u;
    }
    uint32_t all;
    const uint32_t pos0 = block_excl_scan<kLWv>((uint32_t)__popc(word), sh.bs, par, &all);
    for (uint32_t c0 = 0; c0 < all; c0 += kSpList) {
      const uint32_t live = all - c0 < kSpList ? all - c0 : kSpList;
      uint32_t pos = pos0 - c0;  // (mod 2^32: below or beyond this part)
      for (uint32_t m = word; m; m &= m - 1u, ++pos)
        if (pos < kSpList) sh.list[pos] = 32u * tid + ((uint32_t)__ffs(m) - 1u);
      __syncthreads();
      for (uint32_t l0 = 0; l0 < live; l0 += kLT) {
        const uint32_t m = live - l0 < (uint32_t)kLT ? live - l0 : (uint32_t)kLT;
        uint32_t deg = 0, a0 = 0, c = 0, node = 0;
        float cost = 0.0f;
        if (tid < m) {
          node = (uint32_t)(q0 + sh.list[l0 + tid]);
          const uint32_t s = L.n_state[node];
          cost = key_cost((uint32_t)(L.n_pack[node] >> 32));
          const uint4 o0 = g.off[s], o1 = g.off[s + 1];
          a0 = kEps ? o0.y : o0.x;
          deg = kEps ? o1.y - o0.y : o1.x - o0.x;
          if (kEps) {
            c = g.sclass[s];
            if (!kWrite) {  // (every live node of frame t once: its forward-backward sums start at 0)
              L.alpha[node] = 0.0;
              L.beta[node] = 0.0;
            }
          }
        }
        uint32_t tot;
        sh.pre[tid] = block_excl_scan<kLWv>(deg, sh.bs, par, &tot);
        sh.beg[tid] = a0;
        sh.cost[tid] = cost;
        sh.node[tid] = node;
        sh.cls[tid] = c;
        __syncthreads();
        for (uint32_t w0 = 0; w0 < tot; w0 += kLT) {
          const uint32_t it = w0 + tid;
          bool in = false;
          uint32_t j = 0, xb = 0, dn = ~0u, le = kInfKey;
          uint4 r = make_uint4(0, 0, 0, 0);
          if (it < tot) {
            j = search_le(sh.pre, m, it);
            const uint32_t a = sh.beg[j] + (it - sh.pre[j]);
            r = kEps ? g.xarc[a] : g.earc[a];
            dn = sp_lookup<kSpBWin>(L, df, sh.win, r.x);
            if (dn != ~0u) {
              const float exd = key_cost(L.extra_key[dn]);
              const float cd = key_cost((uint32_t)(L.n_pack[dn] >> 32));
              float x = sh.cost[j];
              if (!kEps) x = x + -row[(r.z & 0xffffffu) - 1u];
              x = canon(x + __uint_as_float(r.y));
              xb = __float_as_uint(x);
              const uint32_t xk = cost_key(x);
              le = cost_key(exd + (x - cd));
              in = xk <= cut && xk < kInfKey && le <= lb_key && le < kInfKey;
            }
          }
          uint32_t nsub;
          const uint32_t p = n + block_excl_scan<kLWv>(in ? 1u : 0u, sh.bs, par, &nsub);
          n += nsub;
          if (!kWrite || !in) continue;
          L.links[at + p] = make_uint4(r.w, sh.node[j], dn, xb);
          L.le_key[at + p] = le;
          if (kEps) {
            const uint32_t cl = sh.cls[j];
            L.link_lvl[at + p] = (uint8_t)cl;
            *xmask |= 1u << (cl < 31u ? cl : 31u);
          }
        }
        __syncthreads();
      }
      __syncthreads();
    }
  }
  return n;
}

__device__ __forceinline__ SpFrame sp_dest(const LaneDesc& L, SpLinkShared& sh, int t) {
  const SpFrame f = sp_frame(L, t, kSpBWin);
  __syncthreads();
  for (uint32_t i = threadIdx.x; i < f.m; i += kLT) sh.win[i] = L.n_state[f.n0 + ((uint64_t)i << f.k)];
  __syncthreads();
  return f;
}

union LinkLds {
  LinkShared dense;
  SpLinkShared sparse;
};

// A decode whose forward pass stopped, or whose node store overflowed, gets
// no links (its status already says so).
__device__ __forceinline__ bool links_wanted(const LaneDesc& L) {
  return L.info->status == 0 && (L.info->overflow & kOvfNodes) == 0;
}

// Per frame: emitting links into link_xoff[t], epsilon links into link_end[t]
// (counts; the offset kernel turns them into offsets).
__global__ void __launch_bounds__(kLT) k_links_count(DevGraph g, const LaneDesc* __restrict__ lanes, Params prm) {
  __shared__ LinkLds lds;
  LinkShared& sh = lds.dense;
  const LaneDesc& L = lanes[blockIdx.y];
  if (!links_wanted(L)) return;
  uint32_t par = 0;
  if (sparse_lane(L, prm.flags)) {
    const uint32_t lb_key = cost_key(prm.lattice_beam), ns = slices_of(L, prm.flags);
    for (uint32_t u = blockIdx.x; u < ((uint32_t)L.T + 1u) * ns; u += gridDim.x) {
      const int t = (int)(u / ns);
      const uint32_t k = u % ns;
      uint64_t raw = 0;
      if (!(prm.flags & kFlagSwept) && L.xmask[t] == 0) {
        // a frame whose raw links the forward pass has not counted
        const uint32_t cut = cost_key(L.cut[t]);
        if (t > 0) raw = link_run<false, false>(g, L, sh, par, t, cut, 0, nullptr, nullptr);
        raw += link_run<true, false>(g, L, sh, par, t, cut, 0, nullptr, nullptr);
        __syncthreads();
      }
      const SpFrame f = sp_dest(L, lds.sparse, t);
      const uint32_t ne = t > 0 ? sp_run<false, false>(g, L, lds.sparse, par, t, k, ns, f, lb_key, 0, nullptr) : 0u;
      const uint32_t nx = sp_run<true, false>(g, L, lds.sparse, par, t, k, ns, f, lb_key, 0, nullptr);
      __syncthreads();
      if (threadIdx.x == 0) {
        if (ns > 1) {
          L.slice[(size_t)t * kSlices + k] = make_uint2(ne, nx);
        } else {
          L.link_xoff[t] = ne;
          L.link_end[t] = nx;
        }
        if (raw) atomicAdd((unsigned long long*)&L.info->links, (unsigned long long)raw);
      }
    }
    return;
  }
  // The links found are kept for the write (in the output buffer, free until
  // the final merge), so that it does not gather arcs and log-likelihoods again
  // (a frame's hundred tokens touch most of its 24 KB row): a frame of more than
  // kFound links, or beyond the buffer, is formed twice.
  WD_GLOBAL uint4* const kept = (WD_GLOBAL uint4*)L.out_links;
  const uint64_t cap = L.kept_cap * (sizeof(OutLink) / sizeof(uint4));
  for (int t = (int)blockIdx.x; t <= L.T; t += (int)gridDim.x) {
    const uint32_t cut = cost_key(L.cut[t]);
    const uint32_t ne = t > 0 ? link_run<false, false>(g, L, sh, par, t, cut, 0, nullptr, nullptr, true) : 0u;
    const uint32_t nx = link_run<true, false>(g, L, sh, par, t, cut, ne, nullptr, nullptr, true);
    const uint32_t n = ne + nx;
    __syncthreads();
    if (threadIdx.x == 0)
      sh.base = n <= kFound ? atomicAdd((unsigned long long*)&L.info->found, (unsigned long long)n) : kEmpty;
    __syncthreads();
    const uint64_t base = sh.base;
    const bool fits = n <= kFound && base + n <= cap;
    for (uint32_t i = threadIdx.x; fits && i < n; i += kLT) kept[base + i] = sh.found[i];
    if (threadIdx.x == 0) {
      L.kframe[2 * t] = fits ? base : kEmpty;
      L.link_xoff[t] = ne;
      L.link_end[t] = nx;
      // the step profile's frame record takes the frame's link count
      if (L.prof) {
        uint64_t& rec = L.prof[(size_t)t * kProfSlots + kProfStamps];
        rec = (rec & 0xffffffffull) | ((uint64_t)(ne + nx) << 32);
      }
    }
  }
}

// Per utterance: the frames' link offsets from their counts, the store's
// capacity check and the link totals.
__global__ void __launch_bounds__(kLT) k_links_offsets(const LaneDesc* __restrict__ lanes, Params prm) {
  __shared__ BlockScratch bs;
  const LaneDesc& L = lanes[blockIdx.x];
  if (!links_wanted(L)) return;
  const uint32_t T1 = (uint32_t)L.T + 1;
  const uint32_t per = (T1 + kLT - 1) / kLT;
  const uint32_t f0 = threadIdx.x * per < T1 ? threadIdx.x * per : T1;
  const uint32_t f1 = f0 + per < T1 ? f0 + per : T1;
  uint64_t sum = 0;
  const uint32_t ns = sparse_lane(L, prm.flags) ? slices_of(L, prm.flags) : 1u;
  if (ns > 1)
    // (a slice's counts become what lies before it in its frame's two runs)
    for (uint32_t t = f0; t < f1; ++t) {
      uint2 n = make_uint2(0, 0);
      for (uint32_t k = 0; k < ns; ++k) {
        const uint2 c = L.slice[(size_t)t * kSlices + k];
        L.slice[(size_t)t * kSlices + k] = n;
        n.x += c.x;
        n.y += c.y;
      }
      L.link_xoff[t] = n.x;
      L.link_end[t] = n.y;
      L.xmask[t] = 0;
    }
  for (uint32_t t = f0; t < f1; ++t) sum += L.link_xoff[t] + L.link_end[t];
  uint32_t par = 0;
  uint64_t total;
  uint64_t base = block_excl_scan64<kLWv>(sum, bs, par, &total);
  for (uint32_t t = f0; t < f1; ++t) {
    const uint64_t ne = L.link_xoff[t], nx = L.link_end[t];
    L.link_off[t] = base;
    L.link_xoff[t] = base + ne;
    L.link_end[t] = base + ne + nx;
    base += ne + nx;
  }
  if (threadIdx.x == 0) {
    L.link_off[T1] = total;
    LaneInfo* I = L.info;
    // (a sparse utterance's raw links have been counted; it stores its kept ones)
    if (!sparse_lane(L, prm.flags)) I->links = total;
    I->need_links = total;
    if (total > L.link_cap) {
      I->overflow |= kOvfLinks;
      I->status = 4;  // WD_ECAPACITY
    }
  }
}

// Per frame: the links, at the frame's offsets; the frame's epsilon levels.
__global__ void __launch_bounds__(kLT) k_links_write(DevGraph g, const LaneDesc* __restrict__ lanes, Params prm) {
  __shared__ LinkLds lds;
  LinkShared& sh = lds.dense;
  const LaneDesc& L = lanes[blockIdx.y];
  if (!links_wanted(L)) return;
  uint32_t par = 0, bad = 0;
  if (sparse_lane(L, prm.flags)) {
    const uint32_t lb_key = cost_key(prm.lattice_beam), ns = slices_of(L, prm.flags);
    for (uint32_t u = blockIdx.x; u < ((uint32_t)L.T + 1u) * ns; u += gridDim.x) {
      const int t = (int)(u / ns);
      const uint32_t k = u % ns;
      const SpFrame f = sp_dest(L, lds.sparse, t);
      const uint2 before = ns > 1 ? (uint2)L.slice[(size_t)t * kSlices + k] : make_uint2(0, 0);
      uint32_t xmask = 0;
      if (t > 0) (void)sp_run<false, true>(g, L, lds.sparse, par, t, k, ns, f, lb_key, L.link_off[t] + before.x, &xmask);
      (void)sp_run<true, true>(g, L, lds.sparse, par, t, k, ns, f, lb_key, L.link_xoff[t] + before.y, &xmask);
      const uint32_t all = block_or<kLWv>(xmask, lds.sparse.bs, par);
      if (threadIdx.x == 0) {
        if (ns == 1) L.xmask[t] = all;
        else if (all) (void)atomicOr((uint32_t*)&L.xmask[t], all);
      }
    }
    return;
  }
  const WD_GLOBAL uint4* const kept = (const WD_GLOBAL uint4*)L.out_links;
  for (int t = (int)blockIdx.x; t <= L.T; t += (int)gridDim.x) {
    const uint32_t cut = cost_key(L.cut[t]);
    uint32_t xmask = 0;
    const uint64_t base = L.kframe[2 * t], l0 = L.link_off[t];
    if (base != kEmpty) {
      // the count's records; the destinations found among the frame's nodes
      const uint32_t n = (uint32_t)(L.link_end[t] - l0), ne = (uint32_t)(L.link_xoff[t] - l0);
      const uint64_t d0 = L.node_off[t], d1 = L.node_off[t + 1];
      for (uint32_t i = threadIdx.x; i < n; i += kLT) {
        const uint4 r = kept[base + i];
        const uint64_t dn = node_of(L, d0, d1, r.z);
        if (dn == ~0ull) {
          bad = 1;
          continue;
        }
        L.links[l0 + i] = make_uint4(r.x, r.y, (uint32_t)dn, r.w);
        if (i >= ne) {
          const uint32_t cls = g.sclass[L.n_state[r.y]];
          L.link_lvl[l0 + i] = (uint8_t)cls;
          xmask |= 1u << (cls < 31u ? cls : 31u);
        }
        if (L.n_pack[dn] == pack_tok(cost_key(__uint_as_float(r.w)), r.x)) L.n_pred[dn] = r.y;
      }
    } else {
      if (t > 0) (void)link_run<false, true>(g, L, sh, par, t, cut, l0, &xmask, &bad);
      (void)link_run<true, true>(g, L, sh, par, t, cut, L.link_xoff[t], &xmask, &bad);
    }
    const uint32_t all = block_or<kLWv>(xmask, sh.bs, par);
    if (threadIdx.x == 0) L.xmask[t] = all;
  }
  if (bad) L.info->status = kStatusInternal;
}

void launch_links(const DevGraph& g, const LaneDesc* lanes, int B, const Params& prm, hipStream_t s) {
  const uint32_t blocks = prm.flags & kFlagSwept ? kSliceBlocks : kLinkBlocks;
  hipLaunchKernelGGL(k_links_count, dim3(blocks, B), dim3(kLT), 0, s, g, lanes, prm);
  hipLaunchKernelGGL(k_links_offsets, dim3(B), dim3(kLT), 0, s, lanes, prm);
  hipLaunchKernelGGL(k_links_write, dim3(blocks, B), dim3(kLT), 0, s, g, lanes, prm);
}

}  // namespace wd
