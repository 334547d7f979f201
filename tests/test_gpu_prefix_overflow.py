"""The prefix scan when more pairs pass the prefix than the re-check queue holds.

The queue has 4 B + 65536 slots; a prefix tile whose pairs find no room is
listed with the rest of its slice and settled after the queue.  Which tiles
those are depends on the order of the workgroups, so every answer and every
counter must be the one a queued pair gives: the full filter first, then the
exact re-check.  The inputs stay below the count at which a slice is handed to
the full contraction (d / 16 pairs per 64 queries and 1,024 rows in float16, d
in float32), but for the rows that are there to exceed it.
"""
import math

import numpy as np
import pytest

import oracle
from paper_2608_13144_amd import _lib as L
from paper_2608_13144_amd import api
from gpu_helpers import build_cache, compare_lookup, gpu, host, oracle_cache, say
from test_gpu_prefix import full_contraction, same_answers

pytestmark = pytest.mark.gpu


def slots(B):
    return 4 * B + 65536


# Pairs of a group share the prefix and pass it.  A workgroup's own queue holds
# 512: emptied at the end of a slice (d = 1024: one tile of about 350 pairs; d =
# 128), on the way (d = 512: three tiles of 220) or passed by (float32: 1,300
# pairs a tile).  `stop`: the third tile of eight slices passes whole, so they
# are handed to the full contraction part way.
@pytest.mark.parametrize("prec,B,n,d,groups,store,stop", [
    ("f16", 5000, 40000, 1024, 1500, "f32", False), ("f16", 12000, 131072, 128, 12000, "bf16", False),
    ("f16", 5000, 131072, 512, 2400, "f32", False), ("f16", 5000, 131072, 512, 2400, "f32", True),
    ("f32", 600, 40000, 512, 200, "f32", False),
])
def test_overflow_matches_full(prec, B, n, d, groups, store, stop):
    say("prefix overflow", prec, B, n, d, groups, store, stop)
    rng = np.random.default_rng(B + d)
    lead = 32 if d < 192 else 16
    centre = (20.0 * rng.standard_normal((groups, lead))).astype(np.float32)
    of = rng.integers(0, groups, n)
    z = (0.5 * rng.standard_normal((n, d))).astype(np.float32)
    z[:, :lead] = centre[of]
    # the ball ends in the middle of the group's distances: hits, pairs only
    # the full filter lets through, and pairs it rejects
    r = np.full(n, 0.5 * math.sqrt(2.0 * (d - lead)), np.float32)
    if stop:  # balls that hold every prefix, around rows far off in the other features
        third = (np.arange(n) // 1024 % 3 == 2) & (np.arange(n) < 24 * 1024)
        r[third] = 200.0
        z[third, lead:] += 20.0
    st = oracle_cache(z, rng.integers(0, 5, n).astype(np.int32), r, d, store=store)
    pick = rng.integers(24 * 1024, n, B)
    zq = st.z[pick].copy()
    zq[:, lead:] = 0.5 * rng.standard_normal((B, d - lead)).astype(np.float32)
    size = np.bincount(of, minlength=groups)
    passing = int(size[of[pick]].sum())
    limit = d if prec == "f32" else d // 16
    assert passing > 1.1 * slots(B), (passing, slots(B))
    assert 64 * 1024 / groups < 0.9 * limit
    c = build_cache(st, image=prec == "f16")
    full = full_contraction(c, gpu(zq), L.F32 if prec == "f32" else L.F16)
    for turn in range(2):
        out = c.lookup(gpu(zq), precision=prec, prune=prec == "f16")
        sa, sb = same_answers(out, full, f"overflow {prec} B={B} n={n} d={d}")
        # every pair the full filter passes shares a prefix
        assert sa[L.STAT_RECHECKED] == sb[L.STAT_RECHECKED], (turn, sa.tolist(), sb.tolist())
    assert sa[L.STAT_HITS] > B // 4 and sa[L.STAT_RECHECKED] < passing
    rows = np.arange(0, B, B // 40)
    compare_lookup(out, oracle.lookup_blocked(zq[rows], st.z, st.r, st.label), f"overflow {prec} d={d}", rows)


def few_live(rows, r, n, d):
    """n rows of radius 0 but for `rows`, spread over the cache."""
    rng = np.random.default_rng(n)
    at = np.linspace(500, n - 500, len(rows)).astype(np.int64)
    z = rng.standard_normal((n, d)).astype(np.float32)
    z[at] = rows
    c = api.LipCache(d, n, device="cuda:0", image=False)
    assert c.insert(gpu(z), gpu(np.zeros(n, np.int32)), gpu(np.ones(n, np.float32))) == n
    rr = np.zeros(n, np.float32)
    rr[at] = r
    c.r.copy_(gpu(rr))
    return c


@pytest.mark.parametrize("what", ["band", "norm past float32"])
def test_overflow_goes_through_the_full_filter(what):
    """Pairs the prefix passes and the float32 full filter does not: queries
    opposite to the rows, just outside the ball but within the boundary band
    (the filter's slack is narrower there), and rows whose stored norm is
    infinite.  None of them may count, queued or not."""
    say("prefix overflow, full filter", what)
    rng = np.random.default_rng(4)
    n, d, B = 40000, 96, 2500
    v = rng.standard_normal(d)
    if what == "band":
        rows = (v + 1e-7 * rng.standard_normal((40, d))).astype(np.float32)
        zq = (-v + 1e-7 * rng.standard_normal((B, d))).astype(np.float32)
        dist = np.linalg.norm(rows.astype(np.float64)[:, None] - zq.astype(np.float64)[None], axis=2)
        r = (dist.mean(1) / (1.0 + 0.8e-5)).astype(np.float32)
        off = (dist - r[:, None].astype(np.float64)) / r[:, None]
        assert off.min() > 0.6e-5 and off.max() < 0.97e-5
    else:
        rows = (3.0e18 * np.tile(v, (40, 1))).astype(np.float32)
        zq = np.tile(rows[0], (B, 1))
        r = np.full(40, 1.0e18, np.float32)
        assert (rows.astype(np.float64) ** 2).sum(1).min() > 3.5e38
    assert 40 * B > 1.2 * slots(B)
    c = few_live(rows, r, n, d)
    full = full_contraction(c, gpu(zq), L.F32)
    assert host(full.stats).tolist() == [0, 0, 0, 0]
    for turn in range(2):
        out = c.lookup(gpu(zq), precision="f32")
        same_answers(out, full, what)
