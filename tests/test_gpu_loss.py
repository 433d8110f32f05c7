"""The per-frame loss (Eq. 1 and 2) from the distances it sums, at the edges of its batches of loads: the
double sum of the returned distances, exact to the roundings of a sum of doubles in any order."""
import math

import numpy as np
import pytest

from gpu_helpers import dev, gpu, host, say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T,Na,Nb", [(1, 1, 2), (3, 1023, 1025), (2, 3072, 4096), (2, 4097, 15361),
                                     (1, 16383, 16384), (2, 16385, 20480), (1, 65537, 33000)])
@pytest.mark.parametrize("reduction", [0, 1])
def test_loss_of_the_distances(T, Na, Nb, reduction):
    p = gpu()
    say(f"[loss] {T} x {Na} x {Nb} reduction {reduction}")
    r = np.random.default_rng(Na)
    A, B = (r.uniform(-1, 1, (T, n, 3)).astype(np.float32) for n in (Na, Nb))
    w = r.uniform(.5, 2, T).astype(np.float32)
    g = {k: host(v) for k, v in p.chamfer_fwd(dev(A), dev(B), reduction=reduction,
                                              frame_w=dev(w)).items()}
    for t in range(T):
        sa, sb = (math.fsum(g[k][t].astype(np.float64)) for k in ("dist_a", "dist_b"))
        exp = float(w[t]) * (sa if reduction else sa / Na + sb / Nb)
        # at most a rounding per addition on a path through the sum, and a few more
        assert abs(g["loss"][t] - exp) <= (max(Na, Nb) / 4096 + 24) * 2.0 ** -53 * exp
