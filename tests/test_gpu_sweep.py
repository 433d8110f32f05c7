"""Clouds on which the ordered search's screen settles few queries (Sec. III-A, Eq. 1-2), so that a query wave's
blocks in reach are evaluated for all of its queries at once: targets nearly all as far from the queries, with
and without exact ties, blocks of one repeated point among them, distances beyond what the screen takes, query
waves on two clumps.  Indices and float distances are the oracle's bit for bit."""
import numpy as np
import pytest

import oracle

from gpu_helpers import dev, gpu, host, say

pytestmark = pytest.mark.gpu


def _frame(kind, r, n, m):
    u = r.normal(size=(m, 3))
    B = u / np.linalg.norm(u, axis=1, keepdims=True)
    A = r.normal(size=(n, 3)) * 1e-3
    if kind == "ties":          # every target twice, far from itself in the cloud
        B[m // 2: 2 * (m // 2)] = B[:m // 2]
    elif kind == "repeated":    # whole blocks of one point on the sphere
        B[r.choice(m, m // 2, replace=False)] = B[0]
        B[r.choice(m, m // 4, replace=False)] = B[1]
    elif kind == "beyond":      # squared distances above 1e30, queries within 1e15 of each other
        A, B = A * 1e17, B * 4e15
    elif kind == "clumps":      # query waves that span two clumps, each amid a sphere of targets
        A += 6.0 * r.integers(0, 2, (n, 1))
        B += 6.0 * r.integers(0, 2, (m, 1))
    elif kind == "one query":   # all queries the same point
        A[:] = A[0]
    elif kind == "alike":       # all queries and all targets the same points
        A[:], B[:] = A[0], B[0]
    return A.astype(np.float32), B.astype(np.float32)


# query waves shared by sixteen waves (few of them) and unshared ones
@pytest.mark.parametrize("T,n,m", [(1, 3000, 5000), (12, 6000, 9000), (2, 33000, 20000)])
@pytest.mark.parametrize("kind", ["plain", "ties", "repeated", "beyond", "clumps", "one query", "alike"])
def test_sweep(kind, T, n, m):
    p = gpu()
    say(f"[sweep] {kind} {T} x {n} x {m}")
    r = np.random.default_rng(n + T)
    F = [_frame(kind, r, n, m) for _ in range(T)]
    A, B = np.stack([f[0] for f in F]), np.stack([f[1] for f in F])
    g = {k: host(v) for k, v in p.chamfer_fwd(dev(A), dev(B)).items()}
    for t in {0, T - 1}:
        for Q, P, side in ((A[t], B[t], "a"), (B[t], A[t], "b")):
            some = slice(t, None, 1 + len(Q) // 8000)
            idx, d32, _ = oracle.nearest(Q[some], P)
            assert np.array_equal(g["dist_" + side][t][some].view(np.uint32), d32.view(np.uint32)), side
            assert np.array_equal(g["idx_" + side][t][some], idx), side
