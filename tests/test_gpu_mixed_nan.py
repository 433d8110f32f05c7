"""Points that are NaN on different axes, met in one block of the ordered search (Sec. III-A, Eq. 1-2): none is
a target or stretches a box, so finite queries get the neighbours that the cloud without those points gives
them, with the original indices."""
import numpy as np
import pytest

import oracle
import test_gpu_ordered as ordered

from gpu_helpers import dev, gpu, host, say

pytestmark = pytest.mark.gpu


# query waves shared by 16 waves, unshared ones, and clouds that are ordered in parts
@pytest.mark.parametrize("T,n", [(1, 1500), (60, 1500), (2, 33000)])
@pytest.mark.parametrize("place", ["corner", "spread"])
def test_blocks_of_incomplete_points(place, T, n):
    p = gpu()
    say(f"[mixed nan] {place} {T} x {n}")
    r = np.random.default_rng(n + T)
    A, B = ordered._cloth(r, T, n), ordered._cloth(r, T, n + 100)
    for X in (A, B):
        for t in range(T):
            # a third of the cloud; at the lowest corner their missing coordinates fall into the cell of the
            # others, so whole blocks hold nothing else
            i = r.choice(X.shape[1], X.shape[1] // 3, replace=False)
            if place == "corner":
                X[t, i] = -0.7
            X[t, i, r.integers(0, 3, len(i))] = np.nan
    for two in (True, False):
        kw = {} if two else dict(reduction=1, b_side=False)
        g = {k: host(v) for k, v in p.chamfer_fwd(dev(A), dev(B), **kw).items() if v is not None}
        for t in {0, T - 1}:
            for Q, P, side in ((A[t], B[t], "a"), (B[t], A[t], "b"))[:2 if two else 1]:
                q, c = (np.nonzero(~np.isnan(X).any(1))[0] for X in (Q, P))
                idx, d32, _ = oracle.nearest(Q[q], P[c])
                assert np.array_equal(g["dist_" + side][t][q].view(np.uint32), d32.view(np.uint32)), side
                assert np.array_equal(g["idx_" + side][t][q], c[idx]), side
                rest = np.isnan(Q).any(1)
                assert np.all(np.isinf(g["dist_" + side][t][rest]))
                assert np.all(g["idx_" + side][t][rest] == 0)
