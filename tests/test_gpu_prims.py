"""Sizes at which the device primitives behind graph preparation change path,
checked through the graphs they build (numpy is the reference)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _nd():
    import paper_1704_00386_amd as nd
    return nd


def _numpy_csr(n, src, dst):
    s, d = src.astype(np.int64), dst.astype(np.int64)
    keep = s != d
    s, d = s[keep], d[keep]
    key = np.unique(np.concatenate([s * n + d, d * n + s]))
    off = np.zeros(n + 1, np.int64)
    np.cumsum(np.bincount(key // n, minlength=n), out=off[1:])
    return off, (key % n).astype(np.int32)


# Pairs m: the builder scans 2m flags.  Around one wave row (256), one tile of
# many workgroups (4096), one and two tiles of one workgroup (16384, 32768),
# and the tile count (2048 x 4096) above which tile sums are scanned first.
@pytest.mark.parametrize("m", [0, 1, 2, 127, 128, 129, 2047, 2048, 2049, 8191,
                               8192, 8193, 16383, 16384, 16385, 20479, 40961,
                               (1 << 22) - 1, (1 << 22), (1 << 22) + 1])
def test_csr_at_scan_edges(m):
    import torch
    nd = _nd()
    rng = np.random.default_rng(m + 1)
    n = max(2, m // 6 + 1)
    src = rng.integers(0, n, m).astype(np.int32)
    dst = rng.integers(0, n, m).astype(np.int32)
    ctx = nd.Context(0)
    g = nd.Graph.from_edges(ctx, n, torch.from_numpy(src), torch.from_numpy(dst))
    off, col = g.csr()
    woff, wcol = _numpy_csr(n, src, dst)
    assert np.array_equal(off.cpu().numpy(), woff)
    assert np.array_equal(col.cpu().numpy(), wcol)


# Items n of the partition by sweep bin (one per vertex): around a wave's row,
# a wave's share, one workgroup's 16384 and several; degrees over every bin.
@pytest.mark.parametrize("n", [1, 2, 63, 64, 65, 1023, 1025, 4096, 16383, 16384,
                               16385, 20480, 40001, 200001])
def test_layout_at_partition_edges(n):
    import torch
    nd = _nd()
    rng = np.random.default_rng(n)
    # a few vertices of large degree, many of small, isolated ones at the end
    w = rng.random(6 * n) ** 6
    src = (w * n * 0.9).astype(np.int32)
    dst = rng.integers(0, n, 6 * n).astype(np.int32)
    ctx = nd.Context(0)
    g = nd.Graph.from_edges(ctx, n, torch.from_numpy(src), torch.from_numpy(dst))
    off, col = _numpy_csr(n, src, dst)
    nr, P, _ = g.sizes("core")
    assert (nr, P) == (n, len(col))
    assert np.array_equal(g.sdegree("core").cpu().numpy(), np.diff(off))
    goff, gids = g.incidence("core")
    goff, gids = goff.cpu().numpy(), gids.cpu().numpy()[:, 0]
    assert np.array_equal(goff, off)
    row = np.repeat(np.arange(n), np.diff(off))
    order = np.lexsort((gids, row))
    assert np.array_equal(gids[order], col)
    _, res = g.decompose("core", max_iters=1, allow_not_converged=True)
    assert res["max_sdegree"] == int(np.diff(off).max())


def _random_csr(n, m, seed):
    import torch
    gen = torch.Generator(device="cuda").manual_seed(seed)
    return [torch.randint(0, n, (m,), generator=gen, device="cuda", dtype=torch.int32)
            for _ in range(2)]


def _torch_csr(n, src, dst):
    import torch
    s, d = src.long(), dst.long()
    keep = s != d
    key = torch.unique(torch.cat([s[keep] * n + d[keep], d[keep] * n + s[keep]]))
    off = torch.zeros(n + 1, dtype=torch.int64, device="cuda")
    torch.cumsum(torch.bincount(key // n, minlength=n), 0, out=off[1:])
    return off, (key % n).int()


# The scan of n S-degrees and the partition of n vertices: one workgroup's two
# tiles (32768), the partition's switch to scanned counts (64 tiles of 4096), and
# the tile count (2048 of 4096) above which the scan's tile sums are scanned first.
@pytest.mark.parametrize("n", [32767, 32768, 32769, 64 * 4096, 64 * 4096 + 1,
                               2048 * 4096, 2048 * 4096 + 1])
def test_scan_and_partition_edges(n):
    import torch
    nd = _nd()
    src, dst = _random_csr(n, 3 * n // 2, n)
    g = nd.Graph.from_edges(nd.Context(0), n, src, dst)
    off, col = _torch_csr(n, src, dst)
    goff, gcol = g.csr()
    assert torch.equal(goff.cuda(), off) and torch.equal(gcol.cuda(), col)
    # offsets of the lists in the caller's order, and the lists themselves
    ioff, ids = g.incidence("core")
    assert torch.equal(ioff.cuda(), off)
    row = torch.repeat_interleave(torch.arange(n, device="cuda"), off.diff())
    assert torch.equal(torch.sort(row * n + ids.cuda().flatten().long()).values,
                       row * n + col)


# The sort of 2m keys: one tile of 4096, and 64 tiles, above which its digit
# counts are scanned rather than added up by every workgroup; and the tiles of 2048
# keys whose counts place the distinct ones.
@pytest.mark.parametrize("m", [1023, 1024, 1025, 2048 * 3, 32 * 4096 - 1, 32 * 4096,
                               32 * 4096 + 1])
def test_sort_edges(m):
    import torch
    nd = _nd()
    n = max(2, m // 5)
    src, dst = _random_csr(n, m, m)
    goff, gcol = nd.Graph.from_edges(nd.Context(0), n, src, dst).csr()
    off, col = _torch_csr(n, src, dst)
    assert torch.equal(goff.cuda(), off) and torch.equal(gcol.cuda(), col)
