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
