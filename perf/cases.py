"""The decoder's work, case by case: what a program that uses the library has
it do, from one short command on a small graph to wide-beam lattices and
batches that fill the chip.

A program loads a graph once and then decodes utterance after utterance, so a
state holds the resident graph (one per graph shape, shared by every state of
the process) and the log-likelihoods of its own utterances; one pass is one
whole decode call through the public entry points, results on the host.  The
graphs and log-likelihoods follow the repository's synthetic workloads: Zipf
out-degrees, epsilon arcs that climb levels, exponential weights, and either
peaked log-likelihoods (clean speech: about a hundred tokens a frame) or flat
ones (noise: the max-active limit binds).
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_1804_03243_amd import wfstdec

DEVICE = "cuda:0"

# Graphs: states, arcs, share of epsilon arcs, deepest epsilon chain, pdfs,
# words, mean arc weight.
GRAPHS = {
    "command": dict(S=10_000, A=30_000, eps=0.20, depth=4, P=500, V=1000, w=2.0),
    "hclg": dict(S=5_000_000, A=12_000_000, eps=0.15, depth=4, P=6000, V=30_000, w=3.0),
    "lm": dict(S=30_000_000, A=80_000_000, eps=0.10, depth=4, P=6000, V=100_000, w=3.0),
    "wide": dict(S=2_000_000, A=6_000_000, eps=0.40, depth=8, P=3000, V=30_000, w=3.0),
}


def _case(name, how, graph, B, T0, T1, mean, std, peaks, beam, max_active, lattice_beam, tokens, chunk=0):
    """`how`: the entry point (decode: decode / decode_batch; noalloc:
    wd_decode_noalloc; stream: Stream, then determinize).  Utterance lengths
    are spread over T0..T1; `peaks` is the most peaked pdfs of a frame;
    `tokens` the surviving tokens of a typical frame (for work())."""
    return dict(name=name, how=how, graph=graph, B=B, T0=T0, T1=T1, mean=mean, std=std, peaks=peaks, beam=beam,
                max_active=max_active, lattice_beam=lattice_beam, tokens=tokens, chunk=chunk)


def listed():
    return [
        # a spoken command of two seconds in a serving loop that allocates nothing: the smallest call
        _case("command_60", "noalloc", "command", 1, 60, 60, -12.0, 3.0, 1, 10.0, 2000, 6.0, 150),
        # a whole utterance on the small grammar, as in the smoke check's workload
        _case("grammar_300", "decode", "command", 1, 300, 300, -12.0, 3.0, 1, 10.0, 2000, 6.0, 150),
        # dictation of one utterance on the 5M-state graph: the benchmark's headline call
        _case("dictate_1000", "decode", "hclg", 1, 1000, 1000, -15.0, 4.0, 5, 15.0, 7000, 8.0, 100),
        # the same as it is spoken, a second of audio at a time, then the compact lattice for the client
        _case("stream_700", "stream", "hclg", 1, 700, 700, -15.0, 4.0, 5, 15.0, 7000, 8.0, 100, 32),
        # a large language model: 30M states, 80M arcs
        _case("large_lm_1500", "decode", "lm", 1, 1500, 1500, -15.0, 4.0, 5, 15.0, 10000, 8.0, 130),
        # offline transcription: 64 utterances of ragged lengths, then one utterance for every compute unit
        _case("batch_64", "decode", "hclg", 64, 500, 1500, -15.0, 4.0, 5, 15.0, 7000, 8.0, 100),
        _case("batch_256", "decode", "hclg", 256, 500, 1500, -15.0, 4.0, 5, 15.0, 7000, 8.0, 100),
        # noisy audio: flat log-likelihoods, so max-active is what limits a frame; alone and in a batch
        _case("noisy_333", "decode", "hclg", 1, 333, 333, -8.0, 1.0, 0, 15.0, 7000, 8.0, 7000),
        _case("noisy_batch_48", "decode", "hclg", 48, 100, 400, -8.0, 1.0, 0, 15.0, 7000, 8.0, 7000),
        # wide beams for lattice generation: no limit, and a limit that binds
        _case("wide_800", "decode", "wide", 1, 800, 800, -8.0, 1.0, 0, 20.0, 0, 10.0, 650_000),
        _case("wide_capped_250", "decode", "wide", 1, 250, 250, -8.0, 1.0, 0, 20.0, 50_000, 10.0, 50_000),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["noalloc", "command", "dictate", "dictate", "stream", "batch", "batch", "noisy", "noisy",
                       "noisy_batch", "wide", "capped"])
    if kind in ("noalloc", "command"):
        T = _log_int(rng, 10, 400)
        return _drawn("noalloc" if kind == "noalloc" else "decode", "command", 1, T, T, -12.0, 3.0, 1,
                      rng.choice([8.0, 10.0, 12.0]), rng.choice([500, 2000]), 6.0, 150)
    beam, lat = rng.choice([12.0, 13.0, 15.0, 16.0]), rng.choice([4.0, 6.0, 8.0, 10.0])
    if kind == "dictate":
        T = _log_int(rng, 30, 1500)
        return _drawn("decode", "hclg", 1, T, T, -15.0, 4.0, 5, beam, rng.choice([2000, 7000, 10000]), lat, 100)
    if kind == "stream":
        T = _log_int(rng, 60, 1000)
        return _drawn("stream", "hclg", 1, T, T, -15.0, 4.0, 5, beam, 7000, min(lat, 8.0), 100, _log_int(rng, 8, 64))
    if kind == "batch":
        T = _log_int(rng, 50, 1000)
        return _drawn("decode", "hclg", _log_int(rng, 2, 200), T, T + T // 2, -15.0, 4.0, 5, beam, 7000, lat, 100)
    if kind == "noisy":
        T, ma = _log_int(rng, 20, 400), _log_int(rng, 1000, 20_000)
        return _drawn("decode", rng.choice(["hclg", "wide"]), 1, T, T, -8.0, rng.choice([1.0, 1.5, 2.0]), 0, 15.0,
                      ma, lat, ma)
    if kind == "noisy_batch":
        T, ma = _log_int(rng, 20, 250), _log_int(rng, 1000, 10_000)
        return _drawn("decode", "hclg", _log_int(rng, 2, 48), T, T + T // 2, -8.0, 1.0, 0, 15.0, ma, lat, ma)
    if kind == "wide":
        T = _log_int(rng, 15, 400)
        return _drawn("decode", "wide", 1, T, T, -8.0, 1.0, 0, rng.choice([18.0, 20.0]), 0, 10.0, 500_000)
    T, ma = _log_int(rng, 15, 250), _log_int(rng, 33_000, 200_000)
    return _drawn("decode", "wide", 1, T, T, -8.0, 1.0, 0, 20.0, ma, 10.0, ma)


def _drawn(*a):
    c = _case("", *a)
    del c["name"]
    return c


# ------------------------------------------------------------------ inputs

_graphs: dict = {}  # the process's resident graphs, as a program keeps them: (host arrays, wfstdec.Graph)


def _host_graph(key):
    """Zipf out-degrees on 1..200, epsilon arcs from a state to one of a
    higher level, a self-loop on half of the first arcs; start state 0 fans
    out to 200 arcs; every state is final."""
    c = GRAPHS[key]
    S, A, depth = c["S"], c["A"], c["depth"]
    rng = np.random.Generator(np.random.PCG64([7, S]))
    k = np.arange(1, 201, dtype=np.float64)
    lo, hi = 0.5, 8.0
    for _ in range(100):
        z = 0.5 * (lo + hi)
        p = k ** -z
        lo, hi = (z, hi) if (k * p).sum() / p.sum() > A / S else (lo, z)
    deg = np.searchsorted(np.cumsum(p) / p.sum(), rng.random(S), side="right").clip(0, 199) + 1
    deg[0] = 200
    row = np.zeros(S + 1, np.uint32)
    np.cumsum(deg, out=row[1:])
    n = int(row[-1])
    src = np.repeat(np.arange(S, dtype=np.uint32), deg)
    first = np.zeros(n, bool)
    first[row[:-1]] = True
    level = np.minimum(rng.geometric(0.5, S) - 1, depth).astype(np.int8)
    order = np.argsort(level, kind="stable").astype(np.uint32)  # states by level
    starts = np.searchsorted(level[order], np.arange(depth + 2))
    can = ~first & (level[src] < depth)
    eps = can & (rng.random(n, np.float32) < c["eps"] * n / max(1, int(can.sum())))
    dst = rng.integers(0, S, n, dtype=np.uint32)
    loop = first & (rng.random(n, np.float32) < 0.5) & (deg[src] >= 2) & (src != 0)
    dst[loop] = src[loop]
    e = np.flatnonzero(eps)
    up = level[src[e]] + 1
    to = up + (rng.random(e.size) * (depth + 1 - up)).astype(np.int64)
    a, b = starts[to], starts[to + 1]
    dst[e] = order[np.minimum(a + (rng.random(e.size) * (b - a)).astype(np.int64), b - 1)]
    il = rng.integers(1, c["P"] + 1, n, dtype=np.int32)
    il[eps] = 0
    ol = rng.integers(1, c["V"] + 1, n, dtype=np.int32)
    ol[rng.random(n, np.float32) < 0.9] = 0
    w = rng.standard_exponential(n, np.float32) * np.float32(c["w"])
    return dict(num_states=S, start_state=0, row_ptr=row, dst=dst, ilabel=il, olabel=ol, weight=w, final_weight=None)


def _graph(key):
    if key not in _graphs:
        host = _host_graph(key)
        _graphs[key] = (host, wfstdec.Graph(host, GRAPHS[key]["P"], DEVICE))
    return _graphs[key]


def _lengths(case):
    """B lengths spread evenly over T0..T1, not in order."""
    B, lo, hi = case["B"], case["T0"], case["T1"]
    at = np.random.RandomState(3).permutation(B)
    return [lo + int(round((hi - lo) * int(i) / max(1, B - 1))) for i in at]


def _loglikes(case, seed):
    gen = torch.Generator(device=DEVICE)
    P, out = GRAPHS[case["graph"]]["P"], []
    for b, T in enumerate(_lengths(case)):
        gen.manual_seed(1_000_003 * int(seed) + b)
        x = torch.randn((T, P), generator=gen, device=DEVICE).mul_(case["std"]).add_(case["mean"])
        if case["peaks"]:  # between 3/5 of `peaks` and `peaks` pdfs of a frame stand out
            n = case["peaks"]
            slot = torch.arange(n, device=DEVICE)
            at = torch.randint(P // n, (T, n), generator=gen, device=DEVICE) + slot * (P // n)
            few = torch.randint(max(1, (3 * n) // 5), n + 1, (T, 1), generator=gen, device=DEVICE)
            high = torch.randn((T, n), generator=gen, device=DEVICE).sub_(2.0)
            x.scatter_(1, at, torch.where(slot < few, high, x.gather(1, at)))
        out.append(x)
    return out


def _room(case):
    """Lattice links (and nodes) that the caller's buffers have room for, over
    all utterances: flat log-likelihoods keep tens of links a frame and
    thousands in an utterance's last frames, wide beams thousands a frame."""
    lengths = _lengths(case)
    if case["tokens"] > 20_000:
        return 500_000 + 4000 * sum(lengths)
    if case["peaks"] == 0:
        return sum((32_768 if case["B"] > 1 else 262_144) + 64 * n for n in lengths)
    return sum(4096 + 8 * n for n in lengths)


def _buffers(case):
    """The caller's own arrays, as a serving program keeps them: the outputs
    of every pass on a state land here, zeros behind them."""
    n, frames, B = _room(case), sum(_lengths(case)), case["B"]
    depth = GRAPHS[case["graph"]]["depth"]
    out = dict(count=np.zeros((B, 3), np.int64), cost=np.zeros(B, np.float32),
               words=np.zeros(frames * (depth + 2) + B, np.int32), links=np.zeros(n, wfstdec.LINK_DTYPE),
               nodes=np.zeros(n, wfstdec.NODE_DTYPE))
    if case["how"] == "stream":
        out.update(arcs=np.zeros(4096 + 8 * frames, wfstdec.CLAT_ARC_DTYPE), align=np.zeros(n, np.int32))
    return out


def prepare(case, seed):
    xs, graph = _loglikes(case, seed), _graph(case["graph"])[1]
    state = dict(case=case, graph=graph, xs=xs, args=(case["beam"], case["max_active"], case["lattice_beam"]),
                 out=_buffers(case))
    if case["how"] == "noalloc":
        state["params"] = wfstdec.wd_params(float(case["beam"]), int(case["max_active"]),
                                            float(case["lattice_beam"]), wfstdec.WD_FLAG_ONE_WORKGROUP)
    elif case["how"] == "stream":
        state["chunks"] = list(torch.split(xs[0], case["chunk"]))
    return state


# -------------------------------------------------------------------- a pass

def _copy(out, at, part):
    """part into out[at:], as bytes (large parts with all of torch's threads); the end of it."""
    end = at + len(part)
    if end > len(out):
        raise RuntimeError("a result larger than the caller's buffers: %d of %d" % (end, len(out)))
    if len(part):
        a, b = out[at:end].view(np.uint8), np.ascontiguousarray(part).view(np.uint8)
        if b.size < 1 << 20:
            a[:] = b
        else:
            torch.from_numpy(a).copy_(torch.from_numpy(b))
    return end


def _fields(out):
    """The buffers as plain arrays: a structured one field by field."""
    got = {}
    for k, v in out.items():
        for f in v.dtype.names or (None,):
            x = v if f is None else v[f]
            got[k if f is None else k + "." + f] = x.view(np.int32) if x.dtype == np.uint32 else x
    return got


def run(state):
    case, graph, xs, out = state["case"], state["graph"], state["xs"], state["out"]
    if case["how"] == "noalloc":
        st, cost, nw, stats, _ = wfstdec.wd_decode_noalloc(
            graph.handle, xs[0].data_ptr(), case["T1"], state["params"], None,
            torch.cuda.current_stream().cuda_stream, out["words"], out["links"], out["nodes"])
        if st != wfstdec.WD_OK:
            raise RuntimeError("wd_decode_noalloc: status %d" % st)
        out["cost"][0] = cost
        out["count"][0] = nw, stats["kept_links"], stats["nodes"]
        return _fields(out)
    if case["how"] == "stream":
        s = wfstdec.Stream(graph, 1, case["T1"], *state["args"])
        for x in state["chunks"]:
            s.push([x])
        rs = s.end()
        compact = wfstdec.determinize(rs[0])
        _copy(out["arcs"], 0, compact.arcs)
        _copy(out["align"], 0, compact.align)
    elif case["B"] == 1:
        rs = [wfstdec.decode(graph, xs[0], *state["args"])]
    else:
        rs = wfstdec.decode_batch(graph, xs, *state["args"])
    w = l = n = 0
    for i, r in enumerate(rs):
        out["cost"][i] = r.cost
        out["count"][i] = len(r.words), len(r.links), len(r.nodes)
        w, l, n = _copy(out["words"], w, r.words), _copy(out["links"], l, r.links), _copy(out["nodes"], n, r.nodes)
    return _fields(out)


def work(case):
    """Every log-likelihood once (the decoder refuses NaN wherever it is);
    per frame, for each surviving token its state's two offsets (16 bytes) and
    out-arcs (16 bytes each), and its record (state, cost and predecessor, 12
    bytes) written; two additions and a comparison for each arc."""
    g = GRAPHS[case["graph"]]
    frames, tokens = sum(_lengths(case)), case["tokens"]
    arcs = tokens * g["A"] / g["S"]
    return {"bytes": frames * (4.0 * g["P"] + tokens * 28.0 + arcs * 16.0), "flops": frames * arcs * 3.0}


def tolerance(case):
    """Costs are fp32 sums in an order that the interface fixes, so they are
    the same bit for bit.  Posteriors are sums in 64 bits whose order is free:
    measured 2e-12 from the same sums taken in the log domain (exact() below),
    4e-16 from run to run."""
    return {"rel": 1e-11}


# ---------------------------------------------------- the same in 64 bits

def exact(case, seed):
    """One utterance, token passing over whole frames in numpy with 64-bit
    costs; only the cost where a rounding in 32 bits may decide which links are
    kept."""
    frames = sum(_lengths(case))
    if case["B"] > 1 or case["graph"] == "lm" or frames * case["tokens"] > 3_000_000 or case["tokens"] > 20_000:
        return None
    host = _graphs[case["graph"]][0] if case["graph"] in _graphs else _host_graph(case["graph"])
    L = _loglikes(case, seed)[0].double().cpu().numpy()
    cost, words, links, nodes, close = _viterbi(host, L, case["beam"], case["max_active"], case["lattice_beam"])
    out = {k: None for k in _fields(_buffers(case))}
    out.update(cost=np.array([cost]))
    if close:  # their places may differ
        return out
    room = _room(case)
    for kind, cols in (("links", links), ("nodes", nodes)):
        for f, v in cols.items():
            x = np.zeros(room, np.float64 if v.dtype.kind == "f" else np.int64)
            x[:v.size] = v
            out[kind + "." + f] = x
    out["count"] = np.array([(words.size, links["t"].size, nodes["t"].size)])
    return out


def _arcs_of(host, states, eps):
    """(index into states, arc) of every emitting or epsilon arc out of `states`, in order."""
    row = host["row_ptr"].astype(np.int64, copy=False)
    a0, deg = row[states], row[states + 1] - row[states]
    i = np.repeat(np.arange(states.size), deg)
    arc = np.arange(i.size) - np.repeat(np.cumsum(deg) - deg, deg) + a0[i]
    m = (host["ilabel"][arc] == 0) == eps
    return i[m], arc[m]


def _best_of(state, cost, arc):
    """For each state its smallest (cost, arc)."""
    o = np.lexsort((arc, cost, state))
    s = state[o]
    f = np.ones(s.size, bool)
    f[1:] = s[1:] != s[:-1]
    return s[f], cost[o][f], arc[o][f]


def _viterbi(host, L, beam, max_active, lattice_beam):
    # every array that the frames index is 64-bit once, not once a frame
    host = dict(host, row_ptr=host["row_ptr"].astype(np.int64))
    weight, dst, il = host["weight"], host["dst"], host["ilabel"]
    T = L.shape[0]
    frames = []  # per frame: states, costs, arcs of the surviving tokens
    links = []   # per frame: (source index, arc, cost, dst index, from the frame itself)
    cuts = []
    bound = False  # the max-active limit cut a frame

    def close(s, c, a, cut):
        front = (s, c)
        while front[0].size:
            i, arc = _arcs_of(host, front[0], True)
            x = front[1][i] + weight[arc]
            ok = x <= cut
            d, x, arc = dst[arc[ok]].astype(np.int64), x[ok], arc[ok]
            s2, c2, a2 = _best_of(np.concatenate([s, d]), np.concatenate([c, x]), np.concatenate([a, arc]))
            old = np.full(s2.size, np.inf)
            old[np.searchsorted(s2, s)] = c
            better = c2 < old
            front, (s, c, a) = (s2[better], c2[better]), (s2, c2, a2)
        return s, c, a

    for t in range(T + 1):
        if t == 0:
            s, c, a, cut = np.zeros(1, np.int64), np.zeros(1), np.full(1, -1, np.int64), float(beam)
        else:
            ps, pc, _ = frames[-1]
            ei, ea = _arcs_of(host, ps, False)
            ex = pc[ei] - L[t - 1, il[ea] - 1] + weight[ea]
            s, c, a = _best_of(dst[ea].astype(np.int64), ex, ea)
            cut = c.min() + beam
        s, c, a = close(s, c, a, cut)
        m = c <= cut
        if max_active and m.sum() > max_active:
            cut = min(cut, np.partition(c[m], max_active - 1)[max_active - 1])
            m, bound = c <= cut, True
        s, c, a = s[m], c[m], a[m]
        cuts.append(cut)
        frames.append((s, c, a))
        got = []
        if t:
            k = ex <= cut
            got.append((ei[k], ea[k], ex[k], np.searchsorted(s, dst[ea[k]]), np.zeros(int(k.sum()), bool)))
        xi, xa = _arcs_of(host, s, True)
        xx = c[xi] + weight[xa]
        k = xx <= cut
        got.append((xi[k], xa[k], xx[k], np.searchsorted(s, dst[xa[k]]), np.ones(int(k.sum()), bool)))
        links.append([np.concatenate(v) for v in zip(*got)])
    # extra costs, last frame first; epsilon links until nothing changes
    extra = [np.full(f[0].size, np.inf) for f in frames]
    best = int(np.argmin(frames[T][1]))
    extra[T] = frames[T][1] - frames[T][1][best]
    link_extra = [None] * (T + 1)
    for t in range(T, -1, -1):
        i, arc, x, d, eps = links[t]
        delta = x - frames[t][1][d]
        while True:
            was = extra[t].copy()
            np.minimum.at(extra[t], i[eps], (extra[t][d] + delta)[eps])
            if np.array_equal(was, extra[t]):
                break
        link_extra[t] = extra[t][d] + delta
        if t:
            np.minimum.at(extra[t - 1], i[~eps], link_extra[t][~eps])
    # kept links, posteriors
    keep = [np.isfinite(e) & (e <= lattice_beam) for e in link_extra]
    alpha = [np.full(f[0].size, np.inf) for f in frames]
    beta = [np.full(f[0].size, np.inf) for f in frames]
    alpha[0][np.searchsorted(frames[0][0], 0)] = 0.0
    beta[T][:] = 0.0

    def into(dest, at, v):
        low = np.full(dest.size, np.inf)
        np.minimum.at(low, at, v)
        add = np.zeros(dest.size)
        np.add.at(add, at, np.exp(low[at] - v))
        with np.errstate(divide="ignore", invalid="ignore"):
            new = low - np.log(add)
        hit = add > 0
        dest[hit] = -np.logaddexp(-dest[hit], -new[hit])

    def link_cost(t):
        i, arc, _, d, eps = links[t]
        ac = np.zeros(arc.size)
        if t:
            ac[~eps] = -L[t - 1, il[arc[~eps]] - 1]
        return weight[arc].astype(np.float64) + ac, ac

    def by_depth(t, order):
        """Kept epsilon links of frame t in groups, sources before what they reach."""
        i, _, _, d, eps = links[t]
        k = np.flatnonzero(eps & keep[t])
        dep = np.zeros(frames[t][0].size, np.int64)
        for _ in range(64):
            new = dep.copy()
            np.maximum.at(new, d[k], dep[i[k]] + 1)
            if np.array_equal(new, dep):
                break
            dep = new
        lv = np.unique(dep[i[k]])
        return [k[dep[i[k]] == v] for v in (lv if order > 0 else lv[::-1])]

    for t in range(T + 1):
        i, _, _, d, eps = links[t]
        w = link_cost(t)[0]
        k = np.flatnonzero(~eps & keep[t])
        if k.size:
            into(alpha[t], d[k], alpha[t - 1][i[k]] + w[k])
        for k in by_depth(t, 1):
            into(alpha[t], d[k], alpha[t][i[k]] + w[k])
    for t in range(T, -1, -1):
        i, _, _, d, eps = links[t]
        w = link_cost(t)[0]
        for k in by_depth(t, -1):
            into(beta[t], i[k], beta[t][d[k]] + w[k])
        k = np.flatnonzero(~eps & keep[t])
        if k.size:
            into(beta[t - 1], i[k], beta[t][d[k]] + w[k])
    start = int(np.searchsorted(frames[0][0], 0))
    total = beta[0][start]
    rows, used = [], [np.zeros(f[0].size, bool) for f in frames]
    used[0][start] = True
    for t in range(T + 1):
        i, arc, x, d, eps = links[t]
        w, ac = link_cost(t)
        k = np.flatnonzero(keep[t])
        k = k[np.argsort(arc[k])]
        src = np.where(eps, t, t - 1)[k]
        av = np.array([alpha[u][j] for u, j in zip(src, i[k])])
        ss = np.array([frames[u][0][j] for u, j in zip(src, i[k])], np.int64)
        for u, j in zip(src, i[k]):
            used[u][j] = True
        used[t][d[k]] = True
        rows.append((np.full(k.size, t), arc[k], ss, frames[t][0][d[k]], il[arc[k]], host["olabel"][arc[k]],
                     weight[arc[k]].astype(np.float64), ac[k], x[k], link_extra[t][k],
                     np.exp(total - (av + w[k] + beta[t][d[k]])) if k.size else np.zeros(0)))
    cols = [np.concatenate(v) for v in zip(*rows)]
    words, t, j = [], T, best  # the best path, backwards
    while frames[t][2][j] >= 0:
        arc = frames[t][2][j]
        if host["olabel"][arc]:
            words.append(int(host["olabel"][arc]))
        s = int(np.searchsorted(host["row_ptr"], arc, side="right") - 1)
        t -= int(il[arc] != 0)
        j = int(np.searchsorted(frames[t][0], s))
    ulp = float(np.spacing(np.float32(abs(frames[T][1][best]))))
    # a link this close to the lattice beam, or a kept one to its frame's
    # cutoff, may go the other way in 32 bits (with a max-active limit one
    # token more or less moves the cutoffs of every later frame)
    near = bound or any((np.abs(e - lattice_beam) < 16 * ulp).any() or (v[2][k] > cut - 16 * ulp).any()
                        for e, v, k, cut in zip(link_extra, links, keep, cuts))
    nodes = dict(t=np.concatenate([np.full(int(u.sum()), t) for t, u in enumerate(used)]),
                 state=np.concatenate([f[0][u] for f, u in zip(frames, used)]),
                 cost=np.concatenate([f[1][u] for f, u in zip(frames, used)]),
                 extra=np.concatenate([e[u] for e, u in zip(extra, used)]))
    return (frames[T][1][best], np.array(words[::-1], np.int64), dict(zip(wfstdec.LINK_DTYPE.names, cols)), nodes,
            near)
