"""The sweeps' mappings at the edges of their list-length ranges, with and
without notifications: every SND iterate and the AND result against the CPU
oracle."""
import numpy as np
import pytest

import oracle
from synth import RawGraph

pytestmark = pytest.mark.gpu

# list lengths around one lane, one wave row, a wave's list, a workgroup
EDGES = (1, 4, 5, 15, 16, 17, 63, 64, 65, 255, 256, 257, 511, 513, 1023, 1024,
         1025, 2047, 2048, 2049, 4097, 6500)


def _wheels(rims, per=2, seed=3):
    """Hubs with exactly the given numbers of neighbours: per hub a rim of
    that size whose vertices form a random graph of mean degree about 10, and
    `per` hubs share a rim, so that hubs see each other's rims fall."""
    rng = np.random.default_rng(seed)
    src, dst, base = [], [], 0
    for r in rims:
        hubs = np.arange(base, base + per)
        rim = np.arange(base + per, base + per + r)
        for h in hubs:
            src.append(np.full(r, h))
            dst.append(rim)
        m = 5 * r
        src.append(rng.choice(rim, m))
        dst.append(rng.choice(rim, m))
        base += per + r
    return RawGraph(base, np.concatenate(src).astype(np.int32),
                    np.concatenate(dst).astype(np.int32), "wheels")


def _chain(n, seed):
    """A long ladder hung on a clique: values fall one step per sweep from the
    far end on, for many sweeps with few r-cliques each."""
    i = np.arange(n - 2)
    src = np.concatenate([i, i, np.repeat(np.arange(n, n + 9), 9)])
    dst = np.concatenate([i + 1, i + 2, np.tile(np.arange(n, n + 9), 9)])
    src = np.append(src, [0, 1])
    dst = np.append(dst, [n, n + 1])
    perm = np.random.default_rng(seed).permutation(n + 9)
    return RawGraph(n + 9, perm[src].astype(np.int32), perm[dst].astype(np.int32),
                    "chain")


GRAPHS = {"wheels": lambda: _wheels(EDGES), "wheels1": lambda: _wheels(EDGES, 1, 4),
          "chain": lambda: _chain(700, 2)}
KINDS = {"core": (1, 2), "truss": (2, 3)}


@pytest.mark.parametrize("kind", list(KINDS))
@pytest.mark.parametrize("name", list(GRAPHS))
@pytest.mark.parametrize("switch", ["0", "2", "8"])
def test_iterates_at_list_edges(monkeypatch, name, kind, switch):
    import torch
    import paper_1704_00386_amd as nd
    monkeypatch.setenv("ND_FRONTIER_SWITCH", switch)
    raw = GRAPHS[name]()
    r, s = KINDS[kind]
    og = oracle.Graph.from_raw(raw)
    seq = og.snd(r, s)
    ctx = nd.Context(0)
    g = nd.Graph.from_edges(ctx, raw.n, torch.from_numpy(raw.src),
                            torch.from_numpy(raw.dst))
    for frontier in (False, True):
        its = []
        _, res = g.decompose(kind, "snd", use_frontier=frontier, keep_iterates=its)
        assert res["sweeps"] == len(seq) - 1
        for t, (changed, tau) in enumerate(its, start=1):
            assert np.array_equal(tau.cpu().numpy(), seq[t]), (frontier, t)
            assert changed == int((seq[t] != seq[t - 1]).sum())
        # chunks of sweeps, as without a callback
        kappa, res = g.decompose(kind, "snd", use_frontier=frontier)
        assert np.array_equal(kappa.cpu().numpy(), seq[-1])
        assert res["sweeps"] == len(seq) - 1
        kappa, _ = g.decompose(kind, "and", use_frontier=frontier)
        assert np.array_equal(kappa.cpu().numpy(), seq[-1])


def test_noalloc_without_room_for_support_counts():
    """A decomposition whose flags fit the static workspace while slack words
    and counters do not runs on flags, with the same result."""
    import torch
    import paper_1704_00386_amd as nd
    n = 30_000_000  # 8-bit values: 4 bytes a vertex with flags, 5 without
    small = _chain(700, 5)
    step = n // (small.n + 1)
    src, dst = small.src.astype(np.int64) * step, small.dst.astype(np.int64) * step
    ctx = nd.Context(0)
    g = nd.Graph.from_edges(ctx, n, torch.from_numpy(src.astype(np.int32)),
                            torch.from_numpy(dst.astype(np.int32)))
    g.prepare("core")
    out = torch.full((n,), -1, dtype=torch.int32, device="cuda")
    _, res = g.decompose("core", "snd", use_frontier=True, out=out, noalloc=True)
    want = oracle.Graph.from_raw(small).snd(1, 2)
    assert res["sweeps"] == len(want) - 1 and res["tau_bytes"] == 1
    got = out.cpu().numpy()
    assert np.array_equal(got[np.arange(small.n) * step], want[-1])
    assert int((got != 0).sum()) == int((want[-1] != 0).sum())


# Around the one-workgroup path's limits: 8192 swept r-cliques, 20480
# incidences and lists of 1024; list lengths of every bin inside it; more sweeps than one launch
# runs (the chain), stopped early or not.
def _ring_graph(n, m, seed):
    """n vertices, every one on a cycle, and m further random pairs."""
    rng = np.random.default_rng(seed)
    i = np.arange(n)
    src = np.concatenate([i, rng.integers(0, n, m)])
    dst = np.concatenate([(i + 1) % n, rng.integers(0, n, m)])
    return RawGraph(n, src.astype(np.int32), dst.astype(np.int32), "ring")


TINY = {"ring8191": lambda: _ring_graph(8191, 1900, 1),
        "ring8192": lambda: _ring_graph(8192, 1900, 2),
        "ring8193": lambda: _ring_graph(8193, 1900, 3),
        "entries_below": lambda: _ring_graph(3000, 7200, 4),
        "entries_above": lambda: _ring_graph(3000, 7300, 5),
        "wheels_small": lambda: _wheels((4, 5, 16, 17, 64, 65, 255, 256, 257, 600), 1, 6),
        "hub1024": lambda: _wheels((4, 1024), 1, 8),
        "hub1025": lambda: _wheels((4, 1025), 1, 9),
        "chain": lambda: _chain(700, 7)}


@pytest.mark.parametrize("kind", list(KINDS))
@pytest.mark.parametrize("name", list(TINY))
def test_small_graphs_plain_sweeps(name, kind):
    import torch
    import paper_1704_00386_amd as nd
    raw = TINY[name]()
    r, s = KINDS[kind]
    seq = oracle.Graph.from_raw(raw).snd(r, s)
    ctx = nd.Context(0)
    g = nd.Graph.from_edges(ctx, raw.n, torch.from_numpy(raw.src),
                            torch.from_numpy(raw.dst))
    nsw = int((g.sdegree(kind).cpu().numpy() > 0).sum())
    kappa, res = g.decompose(kind, "snd")
    assert np.array_equal(kappa.cpu().numpy(), seq[-1])
    assert res["sweeps"] == len(seq) - 1
    assert res["updates"] == nsw * res["sweeps"]
    kappa, _ = g.decompose(kind, "and")
    assert np.array_equal(kappa.cpu().numpy(), seq[-1])
    for t in (1, 2, 31, 32, 33, 64, 65):
        if t >= len(seq) - 1:
            break
        tau, res = g.decompose(kind, "snd", max_iters=t, allow_not_converged=True)
        assert res["sweeps"] == t and res["converged"] == 0
        assert np.array_equal(tau.cpu().numpy(), seq[t])
    out = torch.empty(max(len(seq[-1]), 1), dtype=torch.int32, device="cuda")
    g.decompose(kind, "snd", out=out, noalloc=True)
    assert np.array_equal(out.cpu().numpy()[:len(seq[-1])], seq[-1])


# Values narrowed from 32 to 16 to 8 bits between full sweeps: vertices of
# degree about 257 (2^26 gathers a sweep) and hubs of every long list's range,
# whose values fall below 256 within a few sweeps.  Against H-indices by sorting.
def test_values_narrow_between_sweeps():
    import torch
    import paper_1704_00386_amd as nd
    n, m = 1 << 18, (1 << 25) + (1 << 18)
    gen = torch.Generator(device="cuda").manual_seed(11)
    src = torch.randint(0, n, (m,), generator=gen, device="cuda", dtype=torch.int32)
    dst = torch.randint(0, n, (m,), generator=gen, device="cuda", dtype=torch.int32)
    for h, deg in enumerate((300, 900, 1100, 3000, 40000)):
        perm = torch.randperm(n - 5, generator=gen, device="cuda")[:deg] + 5
        src = torch.cat([src, torch.full((deg,), h, device="cuda", dtype=torch.int32)])
        dst = torch.cat([dst, perm.to(torch.int32)])
    ctx = nd.Context(0)
    g = nd.Graph.from_edges(ctx, n, src, dst)
    key = torch.unique(torch.cat([src.long() * n + dst, dst.long() * n + src]))
    key = key[key // n != key % n]
    row, col = key // n, key % n
    off = torch.searchsorted(row, torch.arange(n + 1, device="cuda"))
    rank = torch.arange(row.numel(), device="cuda") - off[row]
    tau = off.diff()
    assert row.numel() >= 1 << 26 and int(tau.max()) >= 32768
    want = []
    for _ in range(6):
        order = torch.sort(row * (1 << 20) + ((1 << 20) - 1 - tau[col])).values
        hits = (((1 << 20) - 1 - (order & ((1 << 20) - 1))) > rank).long()
        total = torch.cat([hits.new_zeros(1), hits.cumsum(0)])
        tau = total[off[1:]] - total[off[:-1]]
        want.append(tau.to(torch.int32))
    assert int(want[0].max()) >= 256 > int(want[-1].max())
    kappa = {}
    for mode in ("snd", "and"):
        for frontier in (False, True):
            if mode == "snd":
                its = []
                g.decompose("core", mode, use_frontier=frontier, max_iters=6,
                            keep_iterates=its, allow_not_converged=True)
                assert [torch.equal(t.cuda().to(torch.int32), w)
                        for (_, t), w in zip(its, want)] == [True] * 6
                for it in (1, 3, 6):
                    t, _ = g.decompose("core", mode, use_frontier=frontier,
                                       max_iters=it, allow_not_converged=True)
                    assert torch.equal(t, want[it - 1])
            kappa[mode, frontier], res = g.decompose("core", mode, use_frontier=frontier)
            assert res["tau_bytes"] == 4
    first = kappa["snd", False]
    assert all(torch.equal(first, k) for k in kappa.values())
    assert torch.equal(g.update("core", first), first)


# The one-workgroup path on a graph most of whose r-cliques are never swept: its
# time follows the swept ones.  A path of 8000 vertices, 4000 sweeps in 125
# launches, alone and among ten million isolated vertices: storing the latter's
# values with every launch takes one workgroup at least 0.13 ms (20 MB at 64
# bytes a clock), 16 ms in all, beside about 20 ms for the sweeps.
def test_small_graph_among_many_isolated_vertices():
    import torch
    import paper_1704_00386_amd as nd
    i = torch.arange(7999, device="cuda", dtype=torch.int32)
    ctx = nd.Context(0)
    ms = {}
    for n in (8000, 10_000_000):
        g = nd.Graph.from_edges(ctx, n, i, i + 1)
        runs = [g.decompose("core", "snd") for _ in range(4)]
        kappa, res = runs[0]
        assert res["sweeps"] == 4000 and int(kappa.sum()) == 8000
        assert int(kappa[8000:].sum()) == 0
        ms[n] = min(r["ms_iterate"] for _, r in runs)
    assert ms[10_000_000] < 1.25 * ms[8000] + 2, ms


# Graphs most of whose lists lie in one range of the longer ones (257..512,
# 513..1024, 1025..2047, above), whose full sweeps may run in launches of their
# own; some lists fall outside the range.
DENSE = {"core_400": ("core", 1300, 0.3, 257, 512), "core_800": ("core", 1300, 0.62, 513, 1024),
         "core_1200": ("core", 1500, 0.82, 1025, 2047),
         "core_mixed": ("core", 1300, 0.79, 800, 1300),
         "core_2200": ("core", 2400, 0.92, 2048, 2400),
         "nucleus13_1400": ("nucleus13", 60, 0.95, 1025, 2047)}


@pytest.mark.parametrize("name", list(DENSE))
def test_long_lists_in_one_range(name):
    import torch
    import paper_1704_00386_amd as nd
    kind, n, p, lo, hi = DENSE[name]
    rng = np.random.default_rng(n)
    i, j = np.triu_indices(n, 1)
    keep = rng.random(i.size) < p
    # and a sparse part
    src = np.concatenate([i[keep], n + np.arange(100)])
    dst = np.concatenate([j[keep], n + 1 + np.arange(100)])
    raw = RawGraph(n + 101, src.astype(np.int32), dst.astype(np.int32), "dense")
    seq = oracle.Graph.from_raw(raw).snd(*nd.RS[kind])
    swept = seq[0][seq[0] > 0]
    assert 2 * ((swept >= lo) & (swept <= hi)).sum() >= swept.size
    ctx = nd.Context(0)
    g = nd.Graph.from_edges(ctx, raw.n, torch.from_numpy(raw.src),
                            torch.from_numpy(raw.dst))
    for frontier in (False, True):
        its = []
        g.decompose(kind, "snd", use_frontier=frontier, keep_iterates=its)
        assert len(its) == len(seq) - 1
        for t, (_, tau) in enumerate(its, start=1):
            assert np.array_equal(tau.cpu().numpy(), seq[t]), (frontier, t)
        for mode in ("snd", "and"):
            kappa, _ = g.decompose(kind, mode, use_frontier=frontier)
            assert np.array_equal(kappa.cpu().numpy(), seq[-1]), (mode, frontier)
    assert np.array_equal(g.update(kind, torch.from_numpy(seq[0])).cpu().numpy(), seq[1])


# A batch with 83200 lists of 1025..2047, so that a tile holds several (a wave
# each) at most tile lengths, and one with few (a workgroup each): the values
# of the graphs one by one.
@pytest.mark.parametrize("count", [2, 64])
def test_batch_of_long_lists(count):
    import torch
    import paper_1704_00386_amd as nd
    n = 1300
    ctx = nd.Context(0)
    i, j = torch.triu_indices(n, n, 1, device="cuda")
    gs = []
    for seed in range(count):
        gen = torch.Generator(device="cuda").manual_seed(seed)
        keep = torch.rand(i.numel(), generator=gen, device="cuda") < 0.84
        gs.append(nd.Graph.from_edges(ctx, n, i[keep].int(), j[keep].int()))
        gs[-1].prepare("core")
        ds = gs[-1].sdegree("core")
        assert int((ds > 1024).sum()) == n
    want = [g.decompose("core", "snd") for g in gs]
    for mode in ("snd", "and"):
        for frontier in (False, True):
            kappas, res = nd.batch_decompose(ctx, gs, "core", mode, use_frontier=frontier)
            for k, r, (w, wr) in zip(kappas, res, want):
                assert torch.equal(k, w), (mode, frontier)
                assert mode == "and" or r["sweeps"] == wr["sweeps"]
