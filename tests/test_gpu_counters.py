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


# few rows against a few thousand targets, one frame and many; the screen's own calls; exhaustive ones
@pytest.mark.parametrize("T,n,m,two,counted", [(1024, 16, 2048, True, True), (256, 384, 8192, False, True),
                                               (1, 16, 2048, False, True), (1, 40000, 64, True, True),
                                               (1024, 512, 256, False, False), (64, 20000, 16, True, False)])
def test_searches_taken(T, n, m, two, counted):
    """The searches of bf16 calls by what they count: every pair evaluated counts no queries."""
    p = gpu()
    r = np.random.default_rng(3)
    A, B = (r.uniform(-.5, .5, (T, k, 3)).astype(np.float32) for k in (n, m))
    st = _stats(p, A, B, **({} if two else dict(reduction=1, b_side=False)))
    assert st["queries"] == (T * (n + m if two else n) if counted else 0)
