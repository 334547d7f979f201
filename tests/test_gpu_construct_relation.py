"""The chunk relation of the de-dup construction: filtered pairs, dense tiles, edges.

``spread`` sets how many candidates lie inside each other's balls: none, a few
per 32 x 32 tile (re-checked one at a time) or nearly all (the tile's float64
sums); ``scale`` moves the rows outside the float16 range, where every pair
passes the filter.
"""
import numpy as np
import pytest

from gpu_helpers import say
from test_gpu_construct import run_both

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,d,spread,scale,store", [
    (1, 32, 1.0, 1.0, "f32"), (33, 96, 0.3, 1.0, "f32"), (1000, 32, 0.05, 1.0, "f32"), (1024, 160, 1.0, 1.0, "bf16"),
    (1025, 64, 0.12, 1.0, "f32"), (2100, 256, 0.5, 1.0, "f32"), (700, 64, 0.12, 1.0e5, "f32"),
    (600, 512, 3.0, 1.0, "bf16"),
])
def test_dedup_relation(n, d, spread, scale, store):
    say("dedup relation", n, d, spread, scale, store)
    rng = np.random.default_rng(n + d)
    centre = rng.standard_normal((7, d))
    z = centre[rng.integers(0, 7, n)] + spread / np.sqrt(d) * rng.standard_normal((n, d))
    z[n // 2:] += 0.2 * rng.standard_normal((n - n // 2, d))
    r = scale * rng.uniform(0.05, 0.4, n)
    run_both((scale * z).astype(np.float32), rng.integers(0, 5, n).astype(np.int32), r.astype(np.float32), d, store=store)


# 1e19 and 1e20: finite features whose squared norm passes the float32 range
@pytest.mark.parametrize("scale", [1.0e18, 1.0e19, 1.0e20])
def test_dedup_norms_past_float32(scale):
    """Near copies within one chunk are duplicates at any finite magnitude."""
    say("dedup norms past float32", scale)
    rng = np.random.default_rng(19)
    n, d = 700, 64
    z = rng.standard_normal((7, d))[rng.integers(0, 7, n)] + 0.12 / np.sqrt(d) * rng.standard_normal((n, d))
    r = (scale * rng.uniform(0.05, 0.4, n)).astype(np.float32)
    _, _, sel = run_both((scale * z).astype(np.float32), rng.integers(0, 5, n).astype(np.int32), r, d)
    assert sel.size < n // 4
