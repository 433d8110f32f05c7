"""The running sums of face areas (Sec. III-B, Eq. 3) where the parallel sum of a chunk of faces begins,
ends or gives way to single additions: bit for bit the oracle's left-to-right sums."""
import numpy as np
import pytest

from gpu_helpers import gpu
from test_gpu_cdf import _check

pytestmark = pytest.mark.gpu


def _mesh(exps, mant, seed):
    """Right triangles of area about 2^exps (exactly where not `mant`), in the given order."""
    r = np.random.default_rng(seed)
    F = len(exps)
    v = np.zeros((1, 3 * F, 3), np.float32)
    h = np.asarray(exps, np.float64) + 1
    a = np.floor(h / 2)
    m = 1 + r.random(F) if mant else np.ones(F)
    v[0, 1::3, 0] = 2.0 ** a
    v[0, 2::3, 1] = m * 2.0 ** (h - a)
    return v, np.arange(3 * F, dtype=np.int32).reshape(F, 3)


@pytest.mark.parametrize("F", [1, 2, 255, 256, 257, 513, 2559, 2560, 2561, 3073, 5119, 5121, 7681])
@pytest.mark.parametrize("kind", ["even", "rough", "zeros"])
def test_sizes(F, kind):
    p = gpu()
    exps = np.full(F, -9) if kind == "even" else np.random.default_rng(F).integers(-12, -6, F)
    v, f = _mesh(exps, kind != "even", F)
    mask = None
    if kind == "zeros":
        mask = (np.random.default_rng(F + 1).random(F) < .4).astype(np.uint8)
        mask[:F // 3] = 0  # zero sums first, over a chunk's edge where the mesh is long
    _check(p, v, f, mask, what=f"{kind} {F}")


@pytest.mark.parametrize("n", [61, 62, 63, 64, 65, 66, 100])
@pytest.mark.parametrize("start", [0, 700, 2555])
def test_single_additions(n, start):
    """n doublings of the sum in one chunk (or over two), around the most that all waves take."""
    p = gpu()
    F = 5200
    exps = np.full(F, -60)
    exps[start:start + n] = np.arange(n) - 50  # each moves the sum to the next binade
    v, f = _mesh(exps, False, n)
    _check(p, v, f, what=f"{n} from {start}")


@pytest.mark.parametrize("every", [2, 37, 41, 2000])
def test_ties_among_others(every):
    """Every `every`th area is half a step of the sum's grid plus whole steps: a tie each."""
    p = gpu()
    F = 5000
    exps = np.full(F, -20)
    exps[0] = 30                # a grid of 2^-22 and, above 2^31, 2^-21
    exps[1::every] = -23
    exps[4000] = 31
    v, f = _mesh(exps, False, every)
    _check(p, v, f, what=f"ties every {every}")


@pytest.mark.parametrize("low,high", [(-140, -130), (100, 110), (-30, 30)])
def test_ranges(low, high):
    p = gpu()
    r = np.random.default_rng(high + 500)
    v, f = _mesh(r.integers(low, high, 6000), True, high + 500)
    _check(p, v, f, what=f"2^{low}..2^{high}")
