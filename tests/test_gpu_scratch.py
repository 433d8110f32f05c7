"""Scratch of the direct calls under a short budget or a refused allocation: the Chamfer search does with less
scratch, gives the same results, and keeps what it has from one call to the next."""
import numpy as np
import pytest

import test_gpu_ordered as ordered

from gpu_helpers import dev, gpu, host, say

pytestmark = pytest.mark.gpu


def _same(x, y):
    for k, v in x.items():
        assert np.array_equal(host(v).view(np.uint8), host(y[k]).view(np.uint8)), k


@pytest.mark.parametrize("precision", [0, 1])
def test_short_budget_allocates_once(precision):
    """A budget with room for the exhaustive search only: after the first call none allocates (an
    allocation would meet the failure that is waiting for it)."""
    p = gpu()
    say(f"[scratch] short budget precision {precision}")
    r = np.random.default_rng(5)
    A, B = (dev(ordered._cloth(r, 40, 4096)) for _ in range(2))
    ref = p.chamfer_fwd(A, B, precision=precision)
    ctx = p.Context(0, hbm_budget_bytes=6 << 20)
    _same(ref, p.chamfer_fwd(A, B, precision=precision, ctx=ctx))
    held = ctx.memory_held()
    ctx.debug_fail_allocs(1)
    out = p.chamfer_fwd(A, B, precision=precision, ctx=ctx)
    _same(ref, out)
    assert ctx.memory_held() == held
    ctx.debug_fail_allocs(0)
    ctx.close()


@pytest.mark.parametrize("T,Na,Nb", [(40, 4096, 4096), (1, 3000, 2000)])
def test_refused_allocation(T, Na, Nb):
    """Where the device refuses the ordered clouds' scratch, the exhaustive search's smaller scratch serves
    the call (one frame of 3,000 x 2,000 needs none); where it refuses that too, the call fails and the next
    one runs."""
    p = gpu()
    say(f"[scratch] refused allocation {T} x {Na} x {Nb}")
    r = np.random.default_rng(6)
    A, B = dev(ordered._cloth(r, T, Na)), dev(ordered._cloth(r, T, Nb))
    ref = p.chamfer_fwd(A, B)
    ctx = p.Context(0)
    ctx.debug_fail_allocs(1)
    _same(ref, p.chamfer_fwd(A, B, ctx=ctx))
    ctx.close()
    if T == 1:
        return
    ctx = p.Context(0)
    ctx.debug_fail_allocs(2)
    with pytest.raises(p.DCError, match="forced"):
        p.chamfer_fwd(A, B, ctx=ctx)
    _same(ref, p.chamfer_fwd(A, B, ctx=ctx))
    ctx.close()
