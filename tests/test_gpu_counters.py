"""The counters of the ordered search: groups of points read again beyond one per query, and queries searched
again although their minimum is met once."""
import numpy as np
import pytest

import test_gpu_ordered as ordered
import test_gpu_sweep as sweep

from gpu_helpers import dev, gpu, say

pytestmark = pytest.mark.gpu


def _stats(p, A, B, **kw):
    ctx = p.Context(0)
    p.chamfer_fwd(dev(A), dev(B), precision=1, ctx=ctx, **kw)
    ctx.sync()
    st = ctx.stats()
    ctx.close()
    say(f"[counters] {st}")
    return st


def test_ordinary_clouds():
    p = gpu()
    r = np.random.default_rng(1)
    T, n = 12, 9000
    st = _stats(p, ordered._cloth(r, T, n), ordered._cloth(r, T, n))
    q = st["queries"]
    assert q == 2 * T * n
    assert q < st["candidates"] < 1.2 * q  # the screen's error leaves some queries two groups, few more
    assert 0 <= st["fallbacks"] < q // 20


def test_queries_the_screen_cannot_settle():
    """Squared distances beyond what the screen takes: every query of the first cloud is searched again."""
    p = gpu()
    r = np.random.default_rng(2)
    T, n, m = 12, 6000, 9000
    F = [sweep._frame("beyond", r, n, m) for _ in range(T)]
    st = _stats(p, np.stack([f[0] for f in F]), np.stack([f[1] for f in F]), reduction=1, b_side=False)
    assert st["queries"] == st["fallbacks"] == T * n
