"""k-truss and (3,4) with lists of exactly the lengths at which the sweeps
change their mapping (one lane, wave rows, a wave's list, a workgroup), beside
short ones that fall in the same sweeps: every SND iterate and the AND result
against the CPU oracle."""
import numpy as np
import pytest

import oracle
from synth import RawGraph

pytestmark = pytest.mark.gpu

LISTS = (255, 256, 257, 512, 513, 1023, 1024, 1025, 2047, 2048, 2049, 4100)
KINDS = {"truss": (2, 3), "nucleus34": (3, 4)}


def _clique_of_hubs(lists, r, seed):
    """len(lists) + r - 1 hubs, all adjacent.  Hub i sees the first l_i minus
    (hubs - r) rim vertices, so an r-set of hubs whose least hub is i (in the
    order of lists) lies in exactly l_i s-cliques."""
    lists = sorted(lists)
    nh = len(lists) + r - 1
    rims = [x - (nh - r) for x in lists] + [lists[-1] - (nh - r)] * (r - 1)
    rim = rims[-1]
    rng = np.random.default_rng(seed)
    src, dst = [], []
    for i in range(nh):
        src.append(np.full(nh - 1 - i, i))
        dst.append(np.arange(i + 1, nh))
        src.append(np.full(rims[i], i))
        dst.append(nh + np.arange(rims[i]))
    i = np.arange(rim)
    width = 1 + 24 * i // rim  # i sees the next `width` ones: the rim peels
    for step in range(1, 26):  # from its thin end on, over many sweeps
        keep = (width >= step) & (i + step < rim)
        src.append(nh + i[keep])
        dst.append(nh + i[keep] + step)
    src.append(nh + rng.integers(0, rim, rim // 8))
    dst.append(nh + rng.integers(0, rim, rim // 8))
    src, dst = np.concatenate(src), np.concatenate(dst)
    perm = rng.permutation(nh + rim)
    return RawGraph(nh + rim, perm[src].astype(np.int32), perm[dst].astype(np.int32),
                    "hubs")


@pytest.mark.parametrize("switch", ["0", "8", None])
@pytest.mark.parametrize("kind", list(KINDS))
def test_lists_of_every_mapping(monkeypatch, kind, switch):
    import torch
    import paper_1704_00386_amd as nd
    if switch is not None:
        monkeypatch.setenv("ND_FRONTIER_SWITCH", switch)
    r, s = KINDS[kind]
    raw = _clique_of_hubs(LISTS, r, 7)
    seq = oracle.Graph.from_raw(raw).snd(r, s)
    # the long lists fall in many sweeps, below values of short ones
    assert set(LISTS) <= set(seq[0].tolist())
    long = seq[0] > 1024
    assert long.sum() >= 4 and len(seq) > 6
    assert seq[-1][long].min() < seq[0][~long].max()
    ctx = nd.Context(0)
    g = nd.Graph.from_edges(ctx, raw.n, torch.from_numpy(raw.src),
                            torch.from_numpy(raw.dst))
    g.prepare(kind)
    for frontier in (False, True):
        its = []
        g.decompose(kind, "snd", use_frontier=frontier, keep_iterates=its)
        assert len(its) == len(seq) - 1
        for t, (_, tau) in enumerate(its, start=1):
            assert np.array_equal(tau.cpu().numpy(), seq[t]), (frontier, t)
        for mode in ("snd", "and", "and", "and"):
            kappa, _ = g.decompose(kind, mode, use_frontier=frontier)
            assert np.array_equal(kappa.cpu().numpy(), seq[-1]), (mode, frontier)
            out = torch.empty(len(seq[-1]), dtype=torch.int32, device="cuda")
            g.decompose(kind, mode, use_frontier=frontier, out=out, noalloc=True)
            assert np.array_equal(out.cpu().numpy(), seq[-1]), (mode, frontier)
        for mode in ("snd", "and"):
            kappas, _ = nd.batch_decompose(ctx, [g, g], kind, mode, use_frontier=frontier)
            assert all(np.array_equal(k.cpu().numpy(), seq[-1]) for k in kappas)


# As the lists shrink: k-truss of G(1000, 1/2), 2^27 gathers a sweep, lists
# around 250 of which the longest start above 255 and fall below, so that the
# values are narrowed from 16 to 8 bits.  The reference applies the update to
# the values themselves (nd_update, which never narrows).
def test_truss_values_narrow():
    import torch
    import paper_1704_00386_amd as nd
    n = 1000
    gen = torch.Generator(device="cuda").manual_seed(5)
    i, j = torch.triu_indices(n, n, 1, device="cuda")
    keep = torch.rand(i.numel(), generator=gen, device="cuda") < 0.5
    ctx = nd.Context(0)
    g = nd.Graph.from_edges(ctx, n, i[keep].int(), j[keep].int())
    g.prepare("truss")
    assert 2 * g.sizes("truss")[1] >= 1 << 26
    tau = g.sdegree("truss").cuda()
    assert int(tau.max()) > 256
    want = []
    for _ in range(6):
        tau = g.update("truss", tau)
        want.append(tau.clone())
    assert int(want[-1].max()) < 256
    kappa = []
    for mode in ("snd", "and"):
        for frontier in (False, True):
            if mode == "snd":
                its = []
                g.decompose("truss", mode, use_frontier=frontier, max_iters=6,
                            keep_iterates=its, allow_not_converged=True)
                assert all(torch.equal(t.cuda(), w) for (_, t), w in zip(its, want))
            k, res = g.decompose("truss", mode, use_frontier=frontier)
            assert res["tau_bytes"] == 2
            kappa.append(k)
    assert all(torch.equal(k, kappa[0]) for k in kappa)
    assert torch.equal(g.update("truss", kappa[0]), kappa[0])
