"""The prefix scan behind the float16 lookup, against the oracle and the full contraction.

A large lookup whose workspace holds the prefix thresholds (or one that asks
for it) scans the first 16 features of every row and re-checks the pairs that
pass; with the plain workspace it runs the full contraction.  Both decide in float64, so every
answer must be the same bit for bit (only the count of re-checked pairs may
fall: the prefix drops pairs the full filter would let through).
"""
import ctypes
import math

import numpy as np
import pytest
import torch

import oracle
from paper_2608_13144_amd import _lib as L
from paper_2608_13144_amd import api
from gpu_helpers import build_cache, compare_lookup, gpu, host, oracle_cache, say

pytestmark = pytest.mark.gpu


def full_contraction(c, zq, prec=L.F16):
    """The lookup on the plain workspace: every pair's whole dot product."""
    lib = L.load()
    B = zq.shape[0]
    need = lib.lipcache_lookup_workspace_bytes(B, c.n, c.d, prec)
    ws = torch.empty(need, dtype=torch.uint8, device=zq.device)
    out = api.LookupResult(torch.empty(B, dtype=torch.int32, device=zq.device),
                           torch.empty(B, dtype=torch.int64, device=zq.device),
                           torch.empty(B, dtype=torch.float32, device=zq.device),
                           torch.empty(4, dtype=torch.int64, device=zq.device),
                           torch.empty(B, dtype=torch.uint8, device=zq.device))
    p = [ctypes.c_void_p(t.data_ptr()) for t in (zq, out.label, out.index, out.dist2, out.stats, out.band, ws)]
    cs = c.cstruct()
    st = lib.lipcache_lookup(ctypes.byref(cs), p[0], B, prec, p[1], p[2], p[3], p[4], p[5], p[6], need,
                             ctypes.c_void_p(torch.cuda.current_stream().cuda_stream))
    assert st == L.OK
    return out


def same_answers(a, b, what):
    for f in ("label", "index", "dist2", "band"):
        x, y = getattr(a, f), getattr(b, f)
        assert torch.equal(x.view(torch.uint8), y.view(torch.uint8)), f"{what}: {f} differs"
    sa, sb = host(a.stats), host(b.stats)
    for k in (L.STAT_HITS, L.STAT_BAND_PAIRS, L.STAT_BAND_QUERIES):
        assert sa[k] == sb[k], f"{what}: stats[{k}] {sa[k]} vs {sb[k]}"
    assert sa[L.STAT_HITS] <= sa[L.STAT_RECHECKED] <= sb[L.STAT_RECHECKED], what
    return sa, sb


def near_queries(rng, st, B, first=0):
    pick = rng.integers(first, st.n, B)
    v = rng.standard_normal((B, st.d))
    v /= np.linalg.norm(v, axis=1, keepdims=True)
    return (st.z[pick].astype(np.float64) + (rng.uniform(0, 2, B) * st.r[pick])[:, None] * v).astype(np.float32)


# B: each number of waves that share 64 queries, and one past it; n: whole
# prefix tiles, one row past a tile, one short; widths with and without padding
@pytest.mark.parametrize("B,n,d,store", [
    (1, 32768, 64, "f32"), (64, 32769, 96, "bf16"), (65, 34815, 256, "f32"), (128, 40961, 160, "f32"),
    (129, 33001, 512, "bf16"), (256, 32768, 768, "f32"), (257, 70001, 64, "bf16"), (513, 33001, 1024, "f32"),
    (1500, 50001, 128, "f32"),
])
def test_prefix_matches_oracle_and_full(B, n, d, store):
    say("prefix scan", B, n, d, store)
    rng = np.random.default_rng(B + n + d)
    z = (2.0 * rng.standard_normal((9, d))[rng.integers(0, 9, n)] + 0.5 * rng.standard_normal((n, d))).astype(np.float32)
    r = rng.uniform(0.05, 0.5, n).astype(np.float32)
    st = oracle_cache(z, rng.integers(0, 9, n).astype(np.int32), r, d, store=store)
    zq = near_queries(rng, st, B)
    c = build_cache(st)
    out = c.lookup(gpu(zq), prune=True)
    what = f"prefix B={B} n={n} d={d} {store}"
    same_answers(out, full_contraction(c, gpu(zq)), what)
    same_answers(out, c.lookup(gpu(zq)), what + " without the option")
    compare_lookup(out, oracle.lookup_blocked(zq, st.z, st.r, st.label), what)


@pytest.mark.parametrize("d,B,part", [(64, 700, 1.0), (256, 700, 0.5), (512, 300, 1.0), (768, 90, 0.5), (1024, 40, 1.0)])
def test_prefix_without_information(d, B, part):
    """Rows that share their first 32 features (all of them, or those of the
    second half, so that slices stop part way): the slices go to the full
    contraction, each pair once."""
    say("prefix without information", d, B, part)
    rng = np.random.default_rng(d + B)
    n = 40000
    z = rng.standard_normal((n, d)).astype(np.float32)
    z[int(n * (1 - part)):, :32] = z[0, :32]
    st = oracle_cache(z, rng.integers(0, 5, n).astype(np.int32), np.full(n, 0.2 * math.sqrt(d), np.float32), d)
    zq = near_queries(rng, st, B, int(n * (1 - part)))
    zq[:, :32] = z[0, :32]
    c = build_cache(st)
    out = c.lookup(gpu(zq), prune=True)
    sa, sb = same_answers(out, full_contraction(c, gpu(zq)), f"d={d} B={B}")
    compare_lookup(out, oracle.lookup_blocked(zq, st.z, st.r, st.label), f"no information d={d} B={B}")
    assert sa[L.STAT_HITS] > B // 4
    # every slice is handed over before a pair is settled
    if part == 1.0:
        assert sa[L.STAT_RECHECKED] == sb[L.STAT_RECHECKED]


# the float32 filter scans 16 features of a float32 store; every size here is
# one that takes the scan by itself
@pytest.mark.parametrize("B,n,d,informative", [
    (60, 200000, 96, True), (700, 70001, 64, True), (130, 40000, 128, True), (600, 33001, 288, True),
    (700, 40000, 64, False), (300, 40000, 512, False),
])
def test_prefix_float32_filter(B, n, d, informative):
    say("prefix float32", B, n, d, informative)
    assert (B + 511) // 512 * 512 * n * (d - 32) >= 2**30
    rng = np.random.default_rng(B + n + d)
    z = rng.standard_normal((n, d)).astype(np.float32)
    if not informative:
        z[:, :16] = z[0, :16]
    st = oracle_cache(z, rng.integers(0, 5, n).astype(np.int32), np.full(n, 0.1 * math.sqrt(d), np.float32), d)
    zq = near_queries(rng, st, B)
    if not informative:
        zq[:, :16] = z[0, :16]
    c = build_cache(st, image=False)
    out = c.lookup(gpu(zq), precision="f32")
    what = f"float32 B={B} n={n} d={d}"
    same_answers(out, full_contraction(c, gpu(zq), L.F32), what)
    compare_lookup(out, oracle.lookup_blocked(zq, st.z, st.r, st.label), what)
    assert host(out.stats)[L.STAT_HITS] > B // 4


def test_prefix_radius_infinite_and_dead():
    """An infinite radius passes every prefix, a radius <= 0 or NaN none."""
    rng = np.random.default_rng(3)
    n, d = 33000, 64
    z = (8.0 * rng.standard_normal((n, d))).astype(np.float32)
    r = np.full(n, 0.5, np.float32)
    lab = rng.integers(0, 5, n).astype(np.int32)
    c = api.LipCache(d, n, device="cuda:0")
    assert c.insert(gpu(z), gpu(lab), gpu(r)) == n
    c.r[777] = math.inf
    c.r[1000:1100] = 0.0
    c.r[1100:1200] = math.nan
    zq = z[[1000, 1100, 5, 32999]] + 0.01
    out = c.lookup(gpu(zq), prune=True)
    assert host(out.index).tolist() == [777, 777, 5, 32999]
    same_answers(out, full_contraction(c, gpu(zq)), "infinite and dead radii")


def test_noalloc_past_the_prefix_workspace():
    """The static workspace holds the plain lookup but not the prefix
    thresholds: the call is served as before, by the full contraction."""
    lib = L.load()
    n, d, B = 4_300_000, 64, 40
    assert lib.lipcache_lookup_workspace_bytes(B, n, d, L.F16) <= L.NOALLOC_SCRATCH_BYTES
    assert lib.lipcache_lookup_workspace_bytes(B, n, d, L.F16 | L.LOOKUP_PRUNE) > L.NOALLOC_SCRATCH_BYTES
    g = torch.Generator(device="cuda:0")
    g.manual_seed(5)
    z = torch.randn(n, d, generator=g, device="cuda:0")
    c = api.LipCache(d, n, device="cuda:0")
    c.insert(z, torch.zeros(n, dtype=torch.int32, device="cuda:0"), torch.full((n,), 1.0, device="cuda:0"))
    zq = (z[:B * 1000:1000] + 0.05).contiguous()
    out = c.lookup_noalloc(zq)
    same_answers(out, c.lookup(zq, prune=True), "noalloc")
    assert host(out.index).tolist() == list(range(0, B * 1000, 1000))
