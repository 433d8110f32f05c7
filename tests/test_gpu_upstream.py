"""What the Chamfer backward (Sec. III-A) does not let into a gradient.  The order of a sum does not depend on
whether the other side's gradient is wanted.  Upstream gradients that are not finite: a frame whose loss gradient is NaN or
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


# rows grouped by small workgroups and targets by large ones, the other way round, and one side sorted
@pytest.mark.parametrize("Na,Nb", [(50000, 40000), (40000, 50000), (140000, 40000)])
def test_order_without_the_other_side(Na, Nb):
    """A row that is the neighbour of 3,000 targets, in terms of magnitudes from 2^-60 to 2^20 that cancel: any
    change of the order shows in the rounding of the sum."""
    p = gpu()
    say(f"[upstream] order {Na} x {Nb}")
    r = np.random.default_rng(Na)
    A = r.uniform(-.5, .5, (1, Na, 3)).astype(np.float32)
    B = r.uniform(-.5, .5, (1, Nb, 3)).astype(np.float32)
    A[0, 77] = 0
    x = np.exp2(r.uniform(-60, 20, (1500, 3))).astype(np.float32)
    hub = r.permutation(Nb)[:3000]
    B[0, hub] = np.concatenate([x, -x])
    ia = r.integers(0, Nb, (1, Na)).astype(np.int32)
    ib = r.integers(0, Na, (1, Nb)).astype(np.int32)
    ib[ib == 77] = 78  # nothing else beside the terms that cancel
    ib[0, hub] = 77
    ia[0, 77] = -1
    one = dev(np.ones(1))
    with_b, without = (p.chamfer_bwd(one, dev(A), dev(B), dev(ia), dev(ib), want_b=w)[0]
                       for w in (True, False))
    assert np.array_equal(host(with_b).view(np.uint32), host(without).view(np.uint32))
