"""Scratch of the direct calls under a short budget or a refused allocation: the Chamfer search does with less
scratch, gives the same results, keeps what it has from one call to the next, and leaves served requests the
room they would have beside the exhaustive search."""
import numpy as np
import pytest

import test_gpu_ordered as ordered

from workloads import gen

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


@pytest.mark.parametrize("over", [0, 1 << 20])
def test_request_beside_the_ordered_clouds(over):
    """A budget for a request, the serving loop and the exhaustive search's scratch, all of whose rest the
    ordered clouds of a direct call take: the request runs, and the direct call again afterwards."""
    p = gpu()
    from paper_2204_03139_amd.serving import Server
    say(f"[scratch] request beside ordered clouds, {over} bytes over")
    r = np.random.default_rng(7)
    A, B = (dev(ordered._cloth(r, 40, 4096)) for _ in range(2))
    held = []
    for budget in (6 << 20, 1 << 30):  # room for the exhaustive search alone, and for any
        ctx = p.Context(0, hbm_budget_bytes=budget)
        ref = p.chamfer_fwd(A, B, ctx=ctx)
        ctx.sync()
        held.append(ctx.memory_held()[0])
        ctx.close()
    verts, faces = gen.trajectory(60, 20, 5)
    obs = ordered._cloth(r, 20, 300)
    need = Server.footprint(verts, faces, obs, 300, precision=0)
    ctx = p.Context(0, hbm_budget_bytes=held[0] + need + (5 << 18) + over)
    assert held[1] > held[0] + (5 << 18) + over
    p.chamfer_fwd(A, B, ctx=ctx)
    srv = Server(ctx)
    for _ in range(2):
        st, loss, _, _ = srv.wait(srv.submit(verts, faces, obs, 300, 5, 0))
        assert st == 0 and np.isfinite(loss).all()
        _same(ref, p.chamfer_fwd(A, B, ctx=ctx))
    assert ctx.memory_held()[0] <= ctx.memory_held()[1]
    srv.close()
