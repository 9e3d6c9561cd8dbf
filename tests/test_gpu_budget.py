"""Device-memory budgets that hold a decomposition with flags but not with
support counts: it runs on flags, with the same result and no error left
behind."""
import ctypes

import numpy as np
import pytest
import torch

import oracle
from synth import RawGraph, chung_lu

pytestmark = pytest.mark.gpu

STEP = 64 << 10


def _smallest(fits, lo, hi):
    """The smallest budget (in STEPs) above lo and up to hi that fits."""
    assert fits(hi)
    while hi - lo > STEP:
        mid = (lo + hi) // (2 * STEP) * STEP
        lo, hi = (lo, mid) if fits(mid) else (mid, hi)
    return hi


class _Case:
    """One graph of n vertices, most of them isolated: the decomposition's
    arrays outweigh the graph's build."""

    def __init__(self, nd, n):
        self.nd, self.n = nd, n
        raw = chung_lu(4000, 2.2, 10.0, seed=9)
        self.raw = raw
        at = np.arange(raw.n, dtype=np.int64) * (n // raw.n)
        self.src = torch.from_numpy(at[raw.src].astype(np.int32)).cuda()
        self.dst = torch.from_numpy(at[raw.dst].astype(np.int32)).cuda()
        want = oracle.Graph.from_raw(raw).peel(1, 2)
        self.want = np.zeros(n, np.int32)
        self.want[at] = want

    def graph(self, ctx):
        g = self.nd.Graph.from_edges(ctx, self.n, self.src, self.dst)
        g.prepare("core")
        return g

    def run(self, budget, host, callback, count_active):
        """kappa, or None when the budget does not hold it."""
        nd = self.nd
        try:
            ctx = nd.Context(0, hbm_budget_bytes=budget)
            g = self.graph(ctx)
        except nd.NdError as e:
            assert e.name == "oom"
            return None
        o, keep = nd._make_opts("snd", use_frontier=True, count_active=count_active,
                                on_iter=(lambda info: 0) if callback else None)
        if host:
            kappa = np.full(self.n, -1, np.int32)
            p = kappa.ctypes.data
        else:
            kappa = torch.full((self.n,), -1, dtype=torch.int32, device="cuda")
            p = kappa.data_ptr()
        st = nd._lib.nd_decompose(g._h, 0, ctypes.byref(o), nd._P(p), int(not host),
                                  nd._stream(), None)
        del keep
        g.close()
        if st == 2:
            return None
        assert st == 0
        return kappa if host else kappa.cpu().numpy()


@pytest.mark.parametrize("host,callback", [(True, False), (False, True), (True, True)])
def test_whatever_holds_flags_runs(nd, host, callback):
    case = _Case(nd, 1 << 20)
    # taking active counts, a decomposition uses flags and never support counts
    least = _smallest(lambda b: case.run(b, host, callback, True) is not None,
                      0, 80 << 20)
    kappa = case.run(least, host, callback, False)
    assert kappa is not None, least
    assert np.array_equal(kappa, case.want)
    assert nd._lib.nd_last_error() == b""


# A batch of eight such graphs in memory for their flags: early members may
# count support, later ones must find room all the same.
@pytest.mark.parametrize("mode", ["snd", "and"])
def test_batch_whatever_holds_flags_runs(nd, mode):
    n, count = 1 << 18, 8
    case = _Case(nd, n)

    def run(budget, frontier):
        try:
            ctx = nd.Context(0, hbm_budget_bytes=budget)
            gs = [case.graph(ctx) for _ in range(count)]
        except nd.NdError as e:
            assert e.name == "oom"
            return None
        try:
            return nd.batch_decompose(ctx, gs, "core", mode, use_frontier=frontier)[0]
        except nd.NdError as e:
            assert e.name == "oom"
            return None

    least = _smallest(lambda b: run(b, False) is not None, 0, 200 << 20)
    # flags: a byte per vertex twice, a stamp per 64 of them, in whole 256 bytes
    flags = count * 2 * (n + n // 64 + 512)
    kappas = run(least + flags, True)
    assert kappas is not None, least
    assert all(np.array_equal(k.cpu().numpy(), case.want) for k in kappas)


# Preparing a k-core takes its arrays and nothing besides that grows with the
# graph (here with room for the 4 bytes a vertex that nd_incidence takes); ego
# estimates 13 bytes a query (id, estimate, sweeps, a mark).
@pytest.mark.parametrize("queries", [0, 400000])
def test_core_in_its_own_arrays(nd, queries):
    n, m = 1 << 17, 1 << 20
    rng = np.random.default_rng(3)
    raw = RawGraph(n, rng.integers(0, n, m).astype(np.int32),
                   rng.integers(0, n, m).astype(np.int32), "random")
    off, col = nd.Graph.from_edges(nd.Context(0), n, torch.from_numpy(raw.src),
                                   torch.from_numpy(raw.dst)).csr()
    nnz = col.numel()
    arrays = 8 * (n + 1) + 8 * nnz + 12 * n + 8 * (n + 1) + 4 * nnz
    ctx = nd.Context(0, hbm_budget_bytes=arrays + (13 * queries or 4 * n) + (192 << 10))
    g = nd.Graph.from_csr(ctx, n, off, col)
    g.prepare("core")
    goff, gids = nd.Graph.incidence(g, "core") if not queries else (None, None)
    if queries:
        qs = rng.integers(0, n, queries)
        est, _ = g.ego_estimate("core", qs)
        some = rng.choice(queries, 200, replace=False)
        want, _ = oracle.Graph.from_raw(raw).ego_estimate(1, 2, qs[some])
        assert np.array_equal(est.cpu().numpy()[some], want)
    else:
        row = np.repeat(np.arange(n), np.diff(goff.cpu().numpy()))
        order = np.lexsort((gids.cpu().numpy()[:, 0], row))
        assert np.array_equal(goff.cpu().numpy(), off.cpu().numpy())
        assert np.array_equal(gids.cpu().numpy()[order, 0], col.cpu().numpy())
    assert nd._lib.nd_last_error() == b""
