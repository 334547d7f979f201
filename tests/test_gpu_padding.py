"""Positions past the batch and rows past the cache never reach the re-check.

The matrix tiles are padded: query positions past the batch (or past a
cluster's list) start at -inf, rows past n carry a threshold of +inf.  Every
count below is exact, so one padded pair let through shows in it.
"""
import numpy as np
import pytest
import torch

from paper_2608_13144_amd import _lib as L
from paper_2608_13144_amd import api
from gpu_helpers import gpu, host, say
from test_gpu_prefix import full_contraction

pytestmark = pytest.mark.gpu


def far_cache(n, d, image=True, store="f32", scale=8.0):
    """Rows far from each other with a radius of 0.5."""
    rng = np.random.default_rng(n + d)
    z = (scale * rng.standard_normal((n, d))).astype(np.float32)
    lab = rng.integers(0, 5, n).astype(np.int32)
    c = api.LipCache(d, n, device="cuda:0", image=image, store=store)
    assert c.insert(gpu(z), gpu(lab), gpu(np.full(n, 0.5, np.float32))) == n
    return c, z, lab


@pytest.mark.parametrize("path,n,d", [
    ("prefix", 33000, 64), ("prefix", 33000, 256), ("full", 33000, 64), ("full", 3000, 512), ("rows", 1500, 96),
    ("rows", 700, 1024), ("f32", 5000, 128), ("f32 prefix", 70001, 96), ("indexed", 20001, 64),
])
def test_unbounded_radius(path, n, d):
    """An infinite radius, and one whose square passes the float32 range: each
    query meets both rows, its own and no other, and has one band pair (the
    infinite radius); a padded position would add pairs."""
    say("unbounded radius", path, n, d)
    c, z, lab = far_cache(n, d, image=path != "rows")
    c.r[77] = np.inf
    c.r[78] = 1.0e20
    own = [5, 600, n - 1]
    zq = gpu(z[own] + np.float32(0.01))
    if path == "prefix":
        res = c.lookup(zq, prune=True)
    elif path == "full":
        res = full_contraction(c, zq)
    elif path == "f32":
        res = full_contraction(c, zq, L.F32)
    elif path == "f32 prefix":
        res = c.lookup(zq, precision="f32")
    elif path == "indexed":
        res, pairs = c.lookup_indexed(c.build_index(16), zq)
        assert pairs >= 3 * 3
    else:
        res = c.lookup(zq)
    assert host(res.index).tolist() == own
    assert host(res.label).tolist() == lab[own].tolist()
    assert host(res.band).tolist() == [1, 1, 1]
    st = host(res.stats)
    assert st[L.STAT_HITS] == 3 and st[L.STAT_RECHECKED] == 9, st.tolist()
    assert st[L.STAT_BAND_PAIRS] == 3 and st[L.STAT_BAND_QUERIES] == 3, st.tolist()


@pytest.mark.parametrize("n,d,B", [(70001, 96, 5), (40003, 128, 600)])
def test_overflowing_products(n, d, B):
    """Finite features past the documented range (products of +inf in the
    float32 filter), the last live row among them: it stands in for the rows
    past n of the last tile.  The spare rows of the cache hold balls around
    everything, so a row past n that is read would be a hit."""
    say("overflowing products", n, d, B)
    assert (B + 511) // 512 * 512 * n * (d - 32) >= 2**30  # takes the prefix scan
    rng = np.random.default_rng(n)
    spare = 1200
    c = api.LipCache(d, n + spare, device="cuda:0", image=False)
    z = rng.standard_normal((n + spare, d)).astype(np.float32)
    z[n - 3:n] = 1.0e18
    r = np.full(n + spare, 0.5, np.float32)
    r[n:] = 1.0e30
    assert c.insert(gpu(z), gpu(np.zeros(n + spare, np.int32)), gpu(r)) == n + spare
    c.n = n
    zq = z[:B] + np.float32(0.001)
    zq[2] = 3.0e20   # q . z overflows against the last rows only
    zq[B - 1] = 3.0e20
    keep = torch.zeros((B + 600, d), device="cuda:0")   # the batch inside a larger allocation
    keep[:B] = gpu(zq)
    q = keep[:B]
    res = c.lookup(q, precision="f32")
    full = full_contraction(c, q, L.F32)
    want = np.arange(B)
    want[[2, B - 1]] = -1
    for what, o in (("prefix", res), ("full", full)):
        assert host(o.index).tolist() == want.tolist(), what
        st = host(o.stats)
        assert st[L.STAT_HITS] == B - 2 and st[L.STAT_BAND_PAIRS] == 0, (what, st.tolist())
