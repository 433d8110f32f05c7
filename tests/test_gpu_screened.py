"""The search over ordered clouds with its blocks screened on the matrix cores (Sec. III-A, Eq. 1-2), which
takes the calls whose query waves fill the chip: the exhaustive search's indices and float distances bit
for bit, on clouds where the screened values decide little (ties, repeated points, clouds far apart or far
from the origin, distances near the ends of the float range, stray and non-finite points)."""
import numpy as np
import pytest

import oracle
import test_gpu_ordered as ordered

from gpu_helpers import dev, gpu, host, say

pytestmark = pytest.mark.gpu


def _frames(kind, r, n, T):
    """T frames of which the first, the middle and the last are of the kind, the others plain cloths."""
    if kind in ("far-origin", "huge", "small", "jumps", "plain"):
        A, B = ordered._cloth(r, 1, n), ordered._cloth(r, 1, n + n // 3)
        if kind == "far-origin":    # coordinates of which only the last bits differ
            A, B = A + np.float32(3000), B + np.float32(3000)
        elif kind == "huge":        # squares near the largest float
            A, B = A * np.float32(2e18), B * np.float32(2e18)
        elif kind == "small":       # squares near the smallest normal float
            A, B = A * np.float32(1e-18), B * np.float32(1e-18)
        elif kind == "jumps":       # clumps apart: query waves that span two of them
            A[0] += r.integers(0, 3, (n, 3)).astype(np.float32) * 5
            B[0] += r.integers(0, 3, (len(B[0]), 3)).astype(np.float32) * 5
    else:
        A, B = ordered._clouds(kind, r, n)
    na, nb = A.shape[1], B.shape[1]
    FA, FB = ordered._cloth(r, T, na), ordered._cloth(r, T, nb)
    for t in (0, T // 2, T - 1):
        FA[t], FB[t] = A[0], B[0]
    return FA, FB


@pytest.mark.parametrize("T,n", [(100, 1500), (12, 17000)])
@pytest.mark.parametrize("kind", ["plain", "far-origin", "huge", "small", "jumps", "padded", "identical",
                                  "lattice", "stray", "far", "line", "tiny", "sphere"])
@pytest.mark.parametrize("two", [True, False])
def test_clouds(kind, T, n, two):
    p = gpu()
    say(f"[screened] {kind} {T} x {n} two {two}")
    A, B = _frames(kind, np.random.default_rng(n + T), n, T)
    kw = {} if two else dict(reduction=1, b_side=False)
    g = {k: host(v) for k, v in p.chamfer_fwd(dev(A), dev(B), **kw).items() if v is not None}
    for t in (0, 1, T - 1):
        for Q, P, side in ((A, B, "a"), (B, A, "b"))[:2 if two else 1]:
            idx, d32, _ = oracle.nearest(Q[t], P[t])
            assert np.array_equal(g["dist_" + side][t].view(np.uint32), d32.view(np.uint32)), (t, side)
            assert np.array_equal(g["idx_" + side][t], idx), (t, side)


# the last query wave and block partly filled, the most lopsided clouds, the largest
@pytest.mark.parametrize("T,Na,Nb", [(2100, 65, 64), (1100, 129, 127), (70, 1921, 7684), (66, 8000, 2000),
                                     (3, 65536, 60001)])
def test_sizes(T, Na, Nb):
    p = gpu()
    say(f"[screened] {T} x {Na} x {Nb}")
    r = np.random.default_rng(Na + Nb)
    A, B = ordered._cloth(r, T, Na), ordered._cloth(r, T, Nb)
    g = {k: host(v) for k, v in p.chamfer_fwd(dev(A), dev(B)).items()}
    for t in (0, T - 1) if Na < 60000 else (T - 1,):
        for Q, P, side in ((A, B, "a"), (B, A, "b")):
            idx, d32, _ = oracle.nearest(Q[t], P[t])
            assert np.array_equal(g["dist_" + side][t].view(np.uint32), d32.view(np.uint32)), (t, side)
            assert np.array_equal(g["idx_" + side][t], idx), (t, side)


@pytest.mark.parametrize("T,n", [(100, 1500), (8, 20000)])
def test_not_finite(T, n):
    ordered.test_not_finite(T, n)
