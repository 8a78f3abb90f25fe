"""Large frames of the one-workgroup mode (frames beyond the LDS token table),
which the leading workgroup runs together with the launch's helpers: against
the CPU oracle at the sizes where that can go wrong."""
import numpy as np
import pytest

import synth
from gpu_compare import assert_same

pytestmark = pytest.mark.gpu


def graph_of(S, A, P, eps, depth, seed):
    cfg = dict(index=900 + seed, family="zipf_levels", S=S, A=A, eps_frac=eps, depth=depth, P=P, V=1000, wmean=2.0)
    rng = np.random.default_rng(seed)
    return synth._pack(synth._graph_zipf_levels(cfg, rng), S)


def flat(T, P, seed, std=1.0):
    return np.random.default_rng(seed).normal(-8.0, std, (T, P)).astype(np.float32)


@pytest.fixture(scope="module")
def wf():
    import torch
    from paper_1804_03243_amd import wfstdec
    assert torch.cuda.is_available()
    return wfstdec


@pytest.fixture(scope="module")
def noisy(wf):
    g = graph_of(60_000, 160_000, 200, 0.25, 5, 1)
    return g, wf.Graph(g, 200)


def check(wf, oracle_mod, g, graph, L, args, mode="workgroup"):
    import torch
    print(f"\n[gpu case] large frames S={g['num_states']} T={L.shape[0]} args={args} mode={mode}", flush=True)
    x, o = torch.from_numpy(L).to(graph.device), oracle_mod.decode(g, L, *args, debug=True)
    # (without the debug outputs the lattice is pruned from the node store)
    assert_same(wf.decode(graph, x, *args, mode=mode), o)
    r = wf.decode(graph, x, *args, debug=True, mode=mode)
    assert_same(r, o, debug=True)
    return r


# no limit; a limit no frame reaches; limits around the LDS table (2048 touched
# states), the tile of 1024 tokens and a cluster's shares; ties at the cutoff
# are kept, so a frame may hold a few more
@pytest.mark.parametrize("mode", ["workgroup", "workgroup_levels"])
@pytest.mark.parametrize("beam,ma", [(14.0, 0), (14.0, 50_000), (12.0, 1023), (12.0, 1025), (13.0, 4097), (9.0, 2047)])
def test_max_active(wf, oracle_mod, noisy, beam, ma, mode):
    g, graph = noisy
    r = check(wf, oracle_mod, g, graph, flat(14, 200, 3), (beam, ma, 6.0), mode)
    assert r.needed["frame_tokens"] > 2048 and r.stats["max_tokens"] >= 1000


def test_in_and_out(wf, oracle_mod, noisy):
    """Flat stretches (large frames) between peaked ones (LDS frames): runs
    open and close several times, on frames of either parity."""
    g, graph = noisy
    L = flat(60, 200, 4)
    rng = np.random.default_rng(5)
    for a, b in ((0, 3), (9, 17), (24, 25), (33, 46)):
        L[a:b] -= 20.0
        for t in range(a, b):
            L[t, rng.choice(200, 3, replace=False)] = -1.0
    r = check(wf, oracle_mod, g, graph, L, (11.0, 3000, 6.0))
    assert r.needed["frame_tokens"] > 2048


@pytest.mark.parametrize("lb", [0.0, 0.5, 30.0, float("inf")])
def test_lattice_beam(wf, oracle_mod, noisy, lb):
    """From the best path alone to every link: one live node a frame, and all
    of them."""
    g, graph = noisy
    check(wf, oracle_mod, g, graph, flat(9, 200, 13), (11.0, 2500, lb))


def test_finals(wf, oracle_mod):
    """Final weights: some states final; then none of the last tokens' states."""
    g = graph_of(30_000, 80_000, 100, 0.2, 4, 3)
    rng = np.random.default_rng(14)
    for share in (0.3, 0.0):
        fw = np.where(rng.random(30_000) < share, rng.exponential(1.0, 30_000), np.inf).astype(np.float32)
        h = dict(g, final_weight=fw)
        check(wf, oracle_mod, h, wf.Graph(h, 100), flat(7, 100, 15), (13.0, 0, 7.0))


def test_ties(wf, oracle_mod):
    """Costs on a grid of 1/16: many equal costs, among them at the limit."""
    g = graph_of(20_000, 60_000, 50, 0.2, 4, 2)
    g["weight"] = synth._quantize(g["weight"])
    graph = wf.Graph(g, 50)
    check(wf, oracle_mod, g, graph, synth._quantize(flat(12, 50, 6)), (10.0, 1500, 5.0))


def test_wide_start(wf, oracle_mod):
    """Frame 0 itself outgrows the LDS table: the start state's epsilon arcs
    reach more states than it has bucket entries."""
    S, fan = 6000, 2500
    src = np.concatenate([np.zeros(fan, np.int64), np.arange(1, S), np.arange(1, fan + 1)])
    dst = np.concatenate([np.arange(1, fan + 1), np.roll(np.arange(1, S), 7), np.arange(1, fan + 1) + fan])
    il = np.concatenate([np.zeros(fan, np.int64), 1 + np.arange(1, S) % 20, np.zeros(fan, np.int64)])
    o = np.argsort(src, kind="stable")
    row = np.zeros(S + 1, np.int64)
    np.cumsum(np.bincount(src, minlength=S), out=row[1:])
    w = np.random.default_rng(8).exponential(0.5, src.size).astype(np.float32)
    g = synth._pack(dict(row_ptr=row, dst=dst[o], ilabel=il[o], olabel=dst[o] % 9, weight=w), S)
    graph = wf.Graph(g, 20)
    for mode in ("workgroup", "workgroup_levels"):
        check(wf, oracle_mod, g, graph, flat(6, 20, 9), (30.0, 0, 8.0), mode)


@pytest.mark.parametrize("B", [3, 9, 40])
def test_batch(wf, oracle_mod, noisy, B):
    """Lanes share the helpers of their XCD; some lanes have no large frame."""
    import torch
    g, graph = noisy
    args = (11.0, 2500, 6.0)
    Ls = [flat(4 + b % 7, 200, 20 + b) for b in range(B)]
    for b in range(0, B, 4):
        Ls[b] -= 10.0
        Ls[b][:, b % 200] = 0.0
    print(f"\n[gpu case] large frames, batch of {B}", flush=True)
    rs = wf.decode_batch(graph, [torch.from_numpy(x).to(graph.device) for x in Ls], *args, mode="workgroup")
    for x, r in zip(Ls, rs):
        assert_same(r, oracle_mod.decode(g, x, *args))


def test_stream(wf, oracle_mod, noisy):
    """Chunks that end inside runs of large frames."""
    import torch
    g, graph = noisy
    L, args = flat(17, 200, 11), (12.0, 3000, 6.0)
    x = torch.from_numpy(L).to(graph.device)
    print("\n[gpu case] large frames, streamed", flush=True)
    s = wf.Stream(graph, 1, 32, *args, mode="workgroup", debug=True)
    for a, b in ((0, 1), (1, 4), (4, 4), (4, 12), (12, 17)):
        s.push([x[a:b]])
    assert_same(s.end()[0], oracle_mod.decode(g, L, *args, debug=True), debug=True)


def test_capacities(wf, oracle_mod, noisy):
    """Per-frame capacities that a large frame outgrows are reported, and the
    retry decodes."""
    import torch
    g, graph = noisy
    L, args = flat(8, 200, 12), (12.0, 3000, 6.0)
    x = torch.from_numpy(L).to(graph.device)
    o = oracle_mod.decode(g, L, *args)
    for caps in (wf.wd_caps(2500, 0, 0, 0, 0, 0), wf.wd_caps(0, 3000, 0, 0, 0, 0), wf.wd_caps(0, 0, 4000, 0, 0, 0)):
        print("\n[gpu case] large frames, small capacities", flush=True)
        with pytest.raises(wf.WdError) as e:
            wf.decode_batch(graph, [x], *args, caps=caps, max_retries=0, mode="workgroup")
        assert e.value.status == wf.WD_ECAPACITY
        assert_same(wf.decode(graph, x, *args, caps=caps, mode="workgroup"), o)


@pytest.mark.parametrize("ma", [120, 200, 320, 500])
def test_link_records(wf, oracle_mod, noisy, ma):
    """Frames with fewer and with more links than a workgroup keeps records of
    (512), of both in one decode; and records beyond the output buffer."""
    import torch
    g, graph = noisy
    L, args = flat(12, 200, 16), (12.0, ma, 6.0)
    r = check(wf, oracle_mod, g, graph, L, args)
    assert r.stats["max_tokens"] < 600
    caps = wf.wd_caps(0, 0, 0, 0, 40, 0)
    assert_same(wf.decode(graph, torch.from_numpy(L).to(graph.device), *args, caps=caps, mode="workgroup"),
                oracle_mod.decode(g, L, *args))


@pytest.mark.parametrize("depth", [2, 3, 4, 9])
@pytest.mark.parametrize("beam,ma", [(11.0, 0), (11.0, 1500)])
def test_chip_wide_levels(wf, oracle_mod, depth, beam, ma):
    """Epsilon levels on both sides of the one from which one launch takes them
    all, and by levels throughout."""
    g = graph_of(20_000, 60_000, 100, 0.3, depth, 30 + depth)
    graph = wf.Graph(g, 100)
    L, args = flat(9, 100, 17), (beam, ma, 6.0)
    check(wf, oracle_mod, g, graph, L, args, "chip")
    import torch
    r = wf.decode(graph, torch.from_numpy(L).to(graph.device), *args, mode="chip", flags=wf.WD_FLAG_EPS_LEVELS)
    assert_same(r, oracle_mod.decode(g, L, *args))


def test_held_results(wf, oracle_mod, noisy):
    """Results stay as they are while later decodes download theirs."""
    import torch
    g, graph = noisy
    Ls = [flat(5, 200, 40 + k) for k in range(6)]
    rs = [wf.decode(graph, torch.from_numpy(x).to(graph.device), 11.0, 2500, 6.0) for x in Ls]
    for x, r in zip(Ls, rs):
        assert_same(r, oracle_mod.decode(g, x, 11.0, 2500, 6.0))


def test_held_results_beyond_the_pool(wf, oracle_mod, noisy):
    """Results of some size kept over more calls than there are pinned blocks
    (leased blocks, then the one they are copied from), small ones among them,
    then batches whose results share a block."""
    import torch
    g, graph = noisy
    lbs = (2.0, 60.0, 60.0, 2.0, 60.0, 60.0, 60.0, 2.0)
    Ls = [flat(6, 200, 70 + k) for k in range(len(lbs))]
    xs = [torch.from_numpy(x).to(graph.device) for x in Ls]
    print("\n[gpu case] held results", flush=True)
    for _ in range(2):  # (the second time on the blocks of the first)
        rs = [wf.decode(graph, x, 11.0, 2500, lb) for x, lb in zip(xs, lbs)]
        sizes = [r.links.nbytes + r.nodes.nbytes + r.words.nbytes for r in rs]
        assert min(sizes) < 64 << 10 < max(sizes) and sorted(sizes)[3] > 64 << 10, sizes
        batches = [wf.decode_batch(graph, xs[k:k + 3], 11.0, 2500, 60.0) for k in range(5)]
        for x, lb, r in zip(Ls, lbs, rs):
            assert_same(r, oracle_mod.decode(g, x, 11.0, 2500, lb))
        for k, b in enumerate(batches):
            for x, r in zip(Ls[k:k + 3], b):
                assert_same(r, oracle_mod.decode(g, x, 11.0, 2500, 60.0))



@pytest.mark.parametrize("beam", [5.0, 9.0, 30.0])
def test_small_frame_capacity(wf, oracle_mod, beam):
    """Frames in LDS are not held to the frame capacity, so their frontiers
    (here of up to 1500 tokens, between a stream's launches and from lane to
    lane) must not reach the arrays behind the ones sized by it."""
    import torch
    g = graph_of(1500, 4200, 50, 0.2, 4, 60)
    graph = wf.Graph(g, 50)
    Ls = [flat(9, 50, 61 + b) for b in range(3)]
    args = (beam, 0, 6.0)
    print(f"\n[gpu case] small frame capacity, beam {beam}", flush=True)
    s = wf.Stream(graph, 3, 16, *args, mode="workgroup", caps=wf.wd_caps(40, 0, 0, 0, 0, 0))
    for a, b in ((0, 2), (2, 3), (3, 9)):
        s.push([torch.from_numpy(x[a:b]).to(graph.device) for x in Ls])
    for x, r in zip(Ls, s.end()):
        o = oracle_mod.decode(g, x, *args)
        assert_same(r, o)
        assert beam < 30.0 or o.stats["max_tokens"] > 1024


@pytest.mark.parametrize("caps", [(2500, 0, 0), (0, 3000, 0), (0, 0, 4000)])
def test_stopped_decode_stats(wf, noisy, caps):
    """A decode that outgrows a capacity reports the same counters every time,
    and no raw links."""
    import torch
    _, graph = noisy
    x = torch.from_numpy(flat(8, 200, 12)).to(graph.device)
    p = wf.wd_params(12.0, 3000, 6.0, wf.WD_FLAG_ONE_WORKGROUP)
    nb, used = wf.wd_workspace_bytes(graph.handle, 1, 8, p, wf.wd_caps(*caps, 0, 0, 0))
    ws = torch.empty(nb + 256, dtype=torch.uint8, device=graph.device)
    seen = []
    print(f"\n[gpu case] large frames, stopped at capacities {caps}", flush=True)
    for _ in range(6):
        st, r = wf.wd_decode(graph.handle, x.data_ptr(), 8, p, used, (ws.data_ptr() + 255) // 256 * 256, nb,
                             torch.cuda.current_stream().cuda_stream)
        assert st == wf.WD_ECAPACITY
        out = wf.wd_result_read(r, False, False)
        wf.wd_result_free(r)
        seen.append((out.stats, out.needed))
    assert seen[0][0]["raw_links"] == 0 and all(s == seen[0] for s in seen[1:]), seen


def hub_graph(S, A, P, hubs, seed):
    """Random arcs; for each (in-degree, share of epsilon arcs) of `hubs` that
    many states' last arcs end in one state (1, 2, ...) instead."""
    rng = np.random.default_rng(seed)
    deg = np.full(S, A // S)
    deg[0] = 64
    row = np.zeros(S + 1, np.int64)
    np.cumsum(deg, out=row[1:])
    n = int(row[-1])
    dst = rng.integers(len(hubs) + 1, S, n)
    il = rng.integers(1, P + 1, n)
    w = rng.exponential(3.0, n).astype(np.float32)
    at = rng.permutation(np.arange(len(hubs) + 1, S))
    for k, (din, eps) in enumerate(hubs):
        a, at = row[at[:din] + 1] - 1, at[din:]
        dst[a] = 1 + k
        il[a[rng.random(a.size) < eps]] = 0
    return synth._pack(dict(row_ptr=row, dst=dst, ilabel=il, olabel=rng.integers(0, 9, n), weight=w), S)


# in-degrees below and above the tokens' out-arcs (the second step's two ways),
# around its smallest (2048 and one more), none; by emitting, by epsilon arcs, by both
@pytest.mark.parametrize("mode", ["workgroup", "chip"])
@pytest.mark.parametrize("hubs,ma", [([(20_000, 0.0)], 2000), ([(20_000, 1.0)], 2000), ([(4000, 0.0), (5000, 1.0)], 3000),
                                     ([(2048, 0.5), (2049, 0.5), (9000, 0.5)], 1500), ([(12_000, 0.5)], 0)])
def test_hubs(wf, oracle_mod, hubs, ma, mode):
    """States that a large share of the graph's arcs end in."""
    g = hub_graph(30_000, 90_000, 60, hubs, 80)
    graph = wf.Graph(g, 60)
    for lb in (6.0, 40.0):
        check(wf, oracle_mod, g, graph, flat(8, 60, 81), (16.0, ma, lb), mode)


def test_many_hubs(wf, oracle_mod):
    """Every live node above the smallest in-degree of a hub, more of them than
    are listed."""
    g = hub_graph(6000, 360_000, 40, [], 82)
    graph = wf.Graph(g, 40)
    for mode in ("workgroup", "chip"):
        check(wf, oracle_mod, g, graph, flat(5, 40, 83), (30.0, 0, 60.0), mode)


@pytest.mark.parametrize("eps", [0.0, 1.0])
def test_hub_time(wf, eps):
    """The pruning of a graph with a state of 400 thousand in-arcs stays within a
    few times that of the raw links (measured 13 times with the in-arcs walked by
    the node)."""
    import torch
    graph = wf.Graph(hub_graph(500_000, 2_000_000, 300, [(400_000, eps)], 84), 300)
    x = torch.from_numpy(flat(30, 300, 85)).to(graph.device)
    print(f"\n[gpu case] hub of 400k in-arcs, eps {eps}", flush=True)
    ms = {}
    for fl in (0, wf.WD_FLAG_NO_INCREMENTAL_PRUNE):
        ms[fl] = min(wf.decode(graph, x, 12.0, 0, 8.0, timing=True, mode="chip", flags=fl).stats["lattice_ms"]
                     for _ in range(4))
    assert ms[0] < 4 * ms[wf.WD_FLAG_NO_INCREMENTAL_PRUNE] + 0.5, ms


@pytest.mark.parametrize("lb", [8.0, 16.0, float("inf")])
def test_wide_lattice_beam_chip(wf, oracle_mod, noisy, lb):
    """Frames whose links are formed in several slices, from a few live nodes
    to all of them."""
    g, graph = noisy
    for T in (3, 11):
        r = check(wf, oracle_mod, g, graph, flat(T, 200, 90), (18.0, 0, lb), "chip")
    assert r.stats["max_tokens"] > 5 * 8192


def test_wide_lattice_time(wf):
    """Where the lattice beam keeps most of a wide decode's last frames, pruning
    from live nodes stays near the raw links' time (measured 5.6 times it with a
    frame's links formed by one workgroup, 1.6 times now)."""
    import torch
    graph = wf.Graph(graph_of(1_000_000, 3_000_000, 300, 0.3, 6, 91), 300)
    x = torch.from_numpy(flat(20, 300, 92)).to(graph.device)
    print("\n[gpu case] wide lattice beam", flush=True)
    ms = {}
    for fl in (0, wf.WD_FLAG_NO_INCREMENTAL_PRUNE):
        ms[fl] = min(wf.decode(graph, x, 20.0, 0, 16.0, timing=True, mode="chip", flags=fl).stats["lattice_ms"]
                     for _ in range(4))
    assert ms[0] < 2.4 * ms[wf.WD_FLAG_NO_INCREMENTAL_PRUNE], ms


def cluster_sizes(r):
    """Workgroups that ran each large frame, by frame (WD_FLAG_PHASES)."""
    large = (r.phases[:, 10] & 1) == 0
    return {int(t): int(r.phases[t, 11] >> 32) for t in np.flatnonzero(large)}


def peaked(T, P, seed):
    L = flat(T, P, seed) - 20.0
    rng = np.random.default_rng(seed)
    for t in range(T):
        L[t, rng.choice(P, 3, replace=False)] = -1.0
    return L.astype(np.float32)


@pytest.mark.parametrize("B,T", [(1, 60), (3, 40), (3, 90), (12, 90)])
def test_cluster_runs_the_frames(wf, oracle_mod, noisy, B, T):
    """Large frames are run by several workgroups: of one utterance, and of
    batches of few and of many frames.  The first run opens while helpers come
    up, so later frames have more of them."""
    import torch
    g, graph = noisy
    Ls, args = [flat(T, 200, 100 + b) for b in range(B)], (11.0, 2500, 6.0)
    print(f"\n[gpu case] cluster sizes, {B} x {T}", flush=True)
    rs = wf.decode_batch(graph, [torch.from_numpy(x).to(graph.device) for x in Ls], *args, mode="workgroup",
                         flags=wf.WD_FLAG_PHASES)
    for x, r in zip(Ls, rs):
        n = cluster_sizes(r)
        print(list(n.items())[:12], max(n.values()))
        assert len(n) > T // 2
        assert max(n.values()) >= (16 if B == 1 else 4), n
        assert max(list(n.values())[8:]) >= list(n.values())[0], n
    assert_same(rs[0], oracle_mod.decode(g, Ls[0], *args))


def test_cluster_for_late_frames(wf, oracle_mod, noisy):
    """Large frames that come after a thousand small ones, and again after a
    hundred, find helpers."""
    import torch
    g, graph = noisy
    L = np.concatenate([peaked(1000, 200, 110), flat(40, 200, 111), peaked(100, 200, 112), flat(40, 200, 113)])
    args = (11.0, 2500, 6.0)
    print("\n[gpu case] late large frames", flush=True)
    r = wf.decode(graph, torch.from_numpy(L).to(graph.device), *args, mode="workgroup", flags=wf.WD_FLAG_PHASES)
    assert_same(r, oracle_mod.decode(g, L, *args))
    n = cluster_sizes(r)
    print(n)
    assert not [t for t in n if t <= 1000], n
    for a in (1000, 1140):
        assert max([v for t, v in n.items() if a < t <= a + 40], default=0) >= 16, n


def test_leaders_alone(wf, oracle_mod, noisy):
    """A batch with an utterance for every compute unit has no helpers: each
    leader runs its large frames alone."""
    import torch
    g, graph = noisy
    B, args = torch.cuda.get_device_properties(0).multi_processor_count, (11.0, 1200, 6.0)
    Ls = [flat(5, 200, 120 + b % 7) for b in range(B)]
    xs = {b: torch.from_numpy(Ls[b]).to(graph.device) for b in range(7)}
    print(f"\n[gpu case] {B} utterances", flush=True)
    rs = wf.decode_batch(graph, [xs[b % 7] for b in range(B)], *args, mode="workgroup", flags=wf.WD_FLAG_PHASES)
    want = [oracle_mod.decode(g, Ls[b], *args) for b in range(7)]
    for b, r in enumerate(rs):
        n = cluster_sizes(r)
        assert n and set(n.values()) == {1}, (b, n)
        assert_same(r, want[b % 7])


def test_concurrent_decodes(wf, oracle_mod, noisy):
    """Utterances on streams and threads of their own, with and without large
    frames.  Helpers of one decode come up late where another's hold the compute
    units, so that runs of large frames open with few and take in more (how often
    is printed: nothing makes sure of it)."""
    import threading
    import torch
    g, graph = noisy
    args = (11.0, 2500, 6.0)
    Ls = [peaked(50, 200, 130), flat(60, 200, 131), flat(60, 200, 132),
          np.concatenate([peaked(30, 200, 133), flat(40, 200, 134)])]
    p = wf.wd_params(*args, wf.WD_FLAG_ONE_WORKGROUP | wf.WD_FLAG_PHASES)
    caps = wf.wd_caps(0, 0, 400_000, 800_000, 400_000, 0)
    got, xs = [[] for _ in Ls], [torch.from_numpy(x).to(graph.device) for x in Ls]
    print("\n[gpu case] concurrent decodes", flush=True)
    want = [oracle_mod.decode(g, x, *args) for x in Ls]

    def run(i):
        T = Ls[i].shape[0]
        nb, used = wf.wd_workspace_bytes(graph.handle, 1, T, p, caps)
        s = torch.cuda.Stream()
        with torch.cuda.stream(s):
            ws = torch.empty(nb + 256, dtype=torch.uint8, device=graph.device)
            for _ in range(8):
                st, r = wf.wd_decode(graph.handle, xs[i].data_ptr(), T, p, used, (ws.data_ptr() + 255) // 256 * 256, nb,
                                     s.cuda_stream)
                got[i].append((st, wf.wd_result_read(r, False, True) if r else None))
                if r:
                    wf.wd_result_free(r)

    torch.cuda.synchronize()
    th = [threading.Thread(target=run, args=(i,)) for i in range(len(Ls))]
    for t in th:
        t.start()
    for t in th:
        t.join()
    for o, rs in zip(want, got):
        for st, r in rs:
            assert st == wf.WD_OK
            assert_same(r, o)
    sizes = [list(cluster_sizes(r).values()) for rs in got for _, r in rs]
    print("decodes with large frames", sum(map(bool, sizes)), "whose cluster grew",
          sum(any(b > a for a, b in zip(n, n[1:])) for n in sizes))


@pytest.mark.parametrize("fan,levels", [(2, 9), (3, 8), (1, 9)])
def test_chip_wide_many_paths(wf, oracle_mod, fan, levels):
    """Graphs with many epsilon paths out of their upper levels (taken by
    levels up to a higher one) and with few."""
    import torch
    S, P = 60_000, 100
    rng = np.random.default_rng(140)
    lvl = rng.integers(0, levels, S)
    lvl[0] = 0
    deg = np.where(lvl < levels - 1, 2 + fan, 2)
    deg[0] = 64 + fan
    row = np.zeros(S + 1, np.int64)
    np.cumsum(deg, out=row[1:])
    n = int(row[-1])
    src = np.repeat(np.arange(S), deg)
    eps = (lvl[src] < levels - 1) & (np.arange(n) - row[src] >= deg[src] - fan)
    dst, il = rng.integers(1, S, n), rng.integers(1, P + 1, n)
    il[eps] = 0
    for l in range(levels - 1):
        k = np.flatnonzero(eps & (lvl[src] == l))
        dst[k] = rng.choice(np.flatnonzero(lvl == l + 1), k.size)
    w = rng.exponential(3.0, n).astype(np.float32)
    g = synth._pack(dict(row_ptr=row, dst=dst, ilabel=il, olabel=rng.integers(0, 9, n), weight=w), S)
    graph = wf.Graph(g, P)
    L = flat(9, P, 141)
    for args in ((13.0, 0, 6.0), (13.0, 6000, 6.0)):
        check(wf, oracle_mod, g, graph, L, args, "chip")
        r = wf.decode(graph, torch.from_numpy(L).to(graph.device), *args, mode="chip", flags=wf.WD_FLAG_EPS_LEVELS)
        assert_same(r, oracle_mod.decode(g, L, *args))
