"""Upstream gradients that are not finite (Chamfer backward, Sec. III-A): a frame whose loss gradient is NaN or
infinite gets no finite gradient and leaves the other frames as they are, also where the unidirectional loss
has no neighbour indices for one side."""
import numpy as np
import pytest

from gpu_helpers import dev, gpu, host, say

pytestmark = pytest.mark.gpu


# sums over listed keys, and over sorted ones
@pytest.mark.parametrize("Na,Nb", [(700, 900), (131100, 64)])
@pytest.mark.parametrize("reduction", [0, 1])
def test_not_finite(reduction, Na, Nb):
    p = gpu()
    say(f"[upstream] {Na} x {Nb} reduction {reduction}")
    r = np.random.default_rng(Na + reduction)
    A = dev(r.uniform(-.5, .5, (3, Na, 3)).astype(np.float32))
    B = dev(r.uniform(-.5, .5, (3, Nb, 3)).astype(np.float32))
    f = p.chamfer_fwd(A, B, reduction=reduction, b_side=reduction == 0)
    ref, got = ([host(g) for g in p.chamfer_bwd(dev(np.array(up)), A, B, f["idx_a"], f["idx_b"],
                                                reduction=reduction, want_b=True)]
                for up in ([1.5, 1.5, 1.5], [np.nan, 1.5, np.inf]))
    for x, y in zip(ref, got):
        assert np.array_equal(x[1].view(np.uint32), y[1].view(np.uint32))
        assert np.isfinite(x).all()
    for t in (0, 2):
        assert not np.isfinite(got[0][t]).any()  # every row of a has its own neighbour
        assert np.isnan(got[1][0]).all()
