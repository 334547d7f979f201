"""Certification through the float16 filter (more than 32 classes, N C d of at least 8e8).

The filter only chooses which classes get an exact float64 logit, so labels
must equal the oracle's and radii, margins and norms its values to float32
rounding (a radius is rounded toward zero, so it may differ by one last place
where the float64 sums differ in order), including rows that the filter leaves
to the float64 kernel: crowded and repeated head rows, rows outside the float16
range and rows that are not finite.
"""
import math

import numpy as np
import pytest

import oracle
from paper_2608_13144_amd import api
from gpu_helpers import gpu, host, say

pytestmark = pytest.mark.gpu

# one float32 last place, and the float64 rounding of d sums (1e-13) beside it
REL = 2.0 ** -23 + 1e-12


def check(z, W, b, store, mode, what, rows=slice(None)):
    sig = oracle.spectral_norm(W).sigma
    ref = oracle.certify(z, W, b, sig, store=store, radius_mode=mode)
    out = api.certify(gpu(z), gpu(W), None if b is None else gpu(b), sig, store=store, radius_mode=mode,
                      want_margin=True, want_norm2=True)
    assert np.array_equal(host(out.label)[rows], ref.label[rows]), f"{what}: labels"
    # a margin is a difference of logits: its float64 error is relative to them
    scale = 1e-13 * np.linalg.norm(z.astype(np.float64), axis=1) * np.linalg.norm(W.astype(np.float64), axis=1).max()
    scale = scale + (0 if b is None else 1e-15 * np.abs(b).max())
    small = np.abs(W.astype(np.float64)[:, None] - W[None]).max(2)
    dmin = np.sqrt((small[small > 0] ** 2).min()) if (small > 0).any() else 1.0
    for name, tol in (("margin", scale), ("r", scale / min(dmin, sig))):
        got, want = host(getattr(out, name)).astype(np.float64), getattr(ref, name).astype(np.float64)
        bad = np.abs(got - want) > REL * np.abs(want) + tol
        bad &= ~((got == want) | (np.isnan(got) & np.isnan(want)))
        assert not bad[rows].any(), f"{what}: {name} {got[rows][bad[rows]][:4]} vs {want[rows][bad[rows]][:4]}"
    n2 = (oracle.bf16_round(z) if store == "bf16" else z).astype(np.float64)
    n2 = (n2 * n2).sum(1)
    assert np.all(np.abs(host(out.norm2)[rows] - n2[rows]) <= REL * n2[rows]), f"{what}: norms"
    return out, ref


# d: each operand width and padded ones; N: whole workgroups of 128 rows, one
# row past, ragged; C: around the 32-class tiles
@pytest.mark.parametrize("N,d,C,store", [
    (760000, 32, 33, "f32"), (196033, 64, 64, "bf16"), (128257, 96, 65, "f32"), (31360, 128, 200, "bf16"),
    (52737, 160, 95, "f32"), (15744, 256, 200, "f32"), (24321, 256, 129, "bf16"), (35840, 320, 70, "f32"),
    (15700, 512, 100, "f32"),
])
@pytest.mark.parametrize("mode", ["conservative", "tight"])
def test_filter_matches_oracle(N, d, C, store, mode):
    if mode == "tight" and N * C > 9_000_000:
        pytest.skip("the tight oracle over this many logits takes minutes")
    say("certify filter", N, d, C, store, mode)
    assert N * C * d >= 8e8
    rng = np.random.default_rng(N + d + C)
    W = (rng.standard_normal((C, d)) / math.sqrt(d)).astype(np.float32)
    b = (0.1 * rng.standard_normal(C)).astype(np.float32)
    mu = 2.0 * rng.standard_normal((C, d))
    z = (mu[rng.integers(0, C, N)] + 0.8 * rng.standard_normal((N, d))).astype(np.float32)
    check(z, W, b, store, mode, f"N={N} d={d} C={C} {store} {mode}")


@pytest.mark.parametrize("mode", ["conservative", "tight"])
def test_filter_leaves_crowded_rows(mode):
    """Near copies of head rows fill the lists, equal rows tie (margin 0, no
    constraint on the tight radius), in some of the rows only."""
    say("certify filter crowded", mode)
    rng = np.random.default_rng(7)
    N, d, C = 104200, 96, 80
    W = (rng.standard_normal((C, d)) / math.sqrt(d)).astype(np.float32)
    W[1:30] = W[0] + (1e-5 * rng.standard_normal((29, d))).astype(np.float32)
    W[41] = W[40]
    z = rng.standard_normal((N, d)).astype(np.float32)
    z[::7] += (6.0 * W[0] / np.linalg.norm(W[0])).astype(np.float32)
    z[3::7] += (6.0 * W[40] / np.linalg.norm(W[40])).astype(np.float32)
    out, ref = check(z, W, None, "f32", mode, f"crowded {mode}")
    assert (ref.margin == 0).sum() > 1000 and (np.asarray(ref.label) < 30).sum() > 5000


def test_filter_leaves_far_rows_and_heads():
    """Rows outside the float16 range, rows that are not finite (no class
    reaches their cut) and a head row outside the range."""
    rng = np.random.default_rng(8)
    N, d, C = 312600, 64, 40
    W = (rng.standard_normal((C, d)) / math.sqrt(d)).astype(np.float32)
    z = rng.standard_normal((N, d)).astype(np.float32)
    z[::50] *= 1.0e5
    z[1::50] = 0.0
    check(z, W, None, "f32", "conservative", "far rows")
    W2 = W.copy()
    W2[5] *= 1.0e6
    check(z, W2, None, "f32", "conservative", "far head row")
    z[2::50, 3] = np.nan
    fine = np.flatnonzero(~np.isnan(z).any(1))
    sig = oracle.spectral_norm(W).sigma
    few = api.certify(gpu(z[:4000]), gpu(W), None, sig)     # float64 kernel for every row
    many = api.certify(gpu(z), gpu(W), None, sig)
    assert np.array_equal(host(few.label), host(many.label)[:4000])
    assert np.array_equal(np.isnan(host(few.r)), np.isnan(host(many.r)[:4000]))
    ref = oracle.certify(z[fine], W, None, sig)
    assert np.array_equal(host(many.label)[fine], ref.label)


def check_rows(z, W, store, mode, rows, what):
    """As check(), with the whole batch on the device and the oracle on `rows` only."""
    sig = oracle.spectral_norm(W).sigma
    ref = oracle.certify(z[rows], W, None, sig, store=store, radius_mode=mode)
    out = api.certify(gpu(z), gpu(W), None, sig, store=store, radius_mode=mode, want_margin=True, want_norm2=True)
    assert np.array_equal(host(out.label)[rows], ref.label), f"{what}: labels"
    scale = 1e-13 * np.linalg.norm(z[rows].astype(np.float64), axis=1) * np.linalg.norm(W.astype(np.float64), axis=1).max()
    apart = np.abs(W.astype(np.float64)[:, None] - W[None]).max(2)
    for name, tol in (("margin", scale), ("r", scale / min(apart[apart > 0].min(), sig))):
        got, want = host(getattr(out, name)).astype(np.float64)[rows], getattr(ref, name).astype(np.float64)
        bad = (np.abs(got - want) > REL * np.abs(want) + tol) & (got != want)
        assert not bad.any(), f"{what}: {name} {got[bad][:4]} vs {want[bad][:4]}"
    n2 = ((oracle.bf16_round(z[rows]) if store == "bf16" else z[rows]).astype(np.float64) ** 2).sum(1)
    assert np.all(np.abs(host(out.norm2)[rows] - n2) <= REL * n2), f"{what}: norms"
    return ref


# the tight radius at every operand width, the narrow ones too (d <= 64 needs
# more logits than the oracle forms in a test: a sample of the rows)
@pytest.mark.parametrize("N,d,C,store", [
    (400033, 32, 64, "f32"), (62503, 64, 200, "bf16"), (192309, 64, 65, "f32"), (63129, 128, 100, "f32"),
    (15744, 256, 200, "bf16"), (15700, 512, 100, "f32"),
])
def test_filter_tight_rows(N, d, C, store):
    say("certify filter tight rows", N, d, C, store)
    assert N * C * d >= 8e8
    rng = np.random.default_rng(N + d + C)
    W = (rng.standard_normal((C, d)) / math.sqrt(d)).astype(np.float32)
    mu = 2.0 * rng.standard_normal((C, d))
    z = (mu[rng.integers(0, C, N)] + 0.8 * rng.standard_normal((N, d))).astype(np.float32)
    rows = np.unique(np.concatenate([np.arange(200), np.arange(N - 200, N), rng.integers(0, N, 3000)]))
    check_rows(z, W, store, "tight", rows, f"tight N={N} d={d} C={C} {store}")


def test_filter_tight_left_rows_past_the_grid():
    """The float64 kernel looks for left rows with 2,048 workgroups of 64 rows:
    past 131,072 rows a workgroup takes a second block.  Left rows in both."""
    say("certify filter tight, left rows past the grid")
    rng = np.random.default_rng(11)
    N, d, C = 180001, 64, 80
    assert N > 2048 * 64
    W = (rng.standard_normal((C, d)) / math.sqrt(d)).astype(np.float32)
    W[1:30] = W[0] + (1e-5 * rng.standard_normal((29, d))).astype(np.float32)
    W[41] = W[40]
    z = rng.standard_normal((N, d)).astype(np.float32)
    left = np.arange(N) % 640 < 5                       # a few blocks in ten, some rows of each
    z[left] += (6.0 * W[0] / np.linalg.norm(W[0])).astype(np.float32)
    rows = np.unique(np.concatenate([np.flatnonzero(left), rng.integers(0, N, 1500), np.arange(N - 100, N)]))
    ref = check_rows(z, W, "f32", "tight", rows, "tight left rows")
    crowded = np.asarray(ref.label) < 30
    assert (crowded & (rows > 2048 * 64)).sum() > 200 and (crowded & (rows < 2048 * 64)).sum() > 500


# masked classes: a large negative bias (it must not reach the error of the
# others) and an infinite one; large biases throughout, where it does
@pytest.mark.parametrize("mode", ["conservative", "tight"])
@pytest.mark.parametrize("mask,spread", [(-1.0e9, 0.1), (-1.0e30, 0.1), (-math.inf, 0.1), (-3.0e3, 300.0)])
def test_filter_masked_classes(mask, spread, mode):
    say("certify filter masked classes", mask, spread, mode)
    rng = np.random.default_rng(12)
    N, d, C = 63129, 128, 100
    W = (rng.standard_normal((C, d)) / math.sqrt(d)).astype(np.float32)
    b = (spread * rng.standard_normal(C)).astype(np.float32)
    b[::9] = mask
    z = (2.0 * rng.standard_normal((N, d))).astype(np.float32)
    rows = np.unique(np.concatenate([np.arange(300), rng.integers(0, N, 2500)]))
    sig = oracle.spectral_norm(W).sigma
    ref = oracle.certify(z[rows], W, b, sig, radius_mode=mode)
    out = api.certify(gpu(z), gpu(W), gpu(b), sig, radius_mode=mode, want_margin=True)
    assert np.array_equal(host(out.label)[rows], ref.label)
    # float64 rounding of sums of this size beside one float32 last place
    tol = 1e-13 * (np.linalg.norm(z[rows].astype(np.float64), axis=1) * 2.0 + 5.0 * spread)
    for name, t in (("margin", tol), ("r", tol / 0.5)):
        got, want = host(getattr(out, name)).astype(np.float64)[rows], getattr(ref, name).astype(np.float64)
        assert np.all(np.abs(got - want) <= REL * np.abs(want) + t), name
    assert not np.isin(host(out.label)[rows], np.arange(0, C, 9)).any()
