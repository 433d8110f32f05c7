"""The nearest-neighbour search over spatially ordered clouds (Sec. III-A, Eq. 1-2): the exhaustive
search's indices and float distances bit for bit, at the edges of its blocks, super-blocks, parts and
wave sharing, on repeated points, ties, stray points and points that are not finite, and where the
budget leaves no room for the ordered clouds."""
import numpy as np
import pytest

import oracle

from gpu_helpers import dev, gpu, host, say, torch

pytestmark = pytest.mark.gpu


def _cloth(r, T, n):
    xy = r.uniform(-.5, .5, (T, n, 2))
    z = 0.05 * np.sin(12 * xy[..., :1]) + 0.05 * np.cos(9 * xy[..., 1:]) + r.normal(0, .005, (T, n, 1))
    return np.concatenate([xy, z], 2).astype(np.float32)


def _check(p, A, B, two=True):
    T = A.shape[0]
    kw = {} if two else dict(reduction=1, b_side=False)
    g = p.chamfer_fwd(dev(A), dev(B), **kw)
    torch.cuda.synchronize()
    for t in range(T):
        for q, c, side in ((A, B, "a"), (B, A, "b"))[:2 if two else 1]:
            idx, d32, _ = oracle.nearest(q[t], c[t])
            assert np.array_equal(host(g["idx_" + side])[t], idx), (t, side)
            assert np.array_equal(host(g["dist_" + side])[t].view(np.uint32), d32.view(np.uint32)), \
                (t, side)


# points around a block (32), a query wave (64), a super-block (2,048), the largest cloud of one
# workgroup (16,384) and a part of a larger one; frames that share query waves between 16, 4 and 1
# waves (16 below 512 query waves on a side, 4 up to 1,024 among more than 16,384 targets)
@pytest.mark.parametrize("T,Na,Nb", [
    (1, 64, 64), (2, 65, 127), (1, 257, 2047), (1, 2049, 4095), (12, 2112, 2100), (40, 3333, 3400),
    (1, 512, 20000), (3, 9000, 1500), (1, 16384, 16384), (1, 16385, 16383), (2, 33000, 24577),
    (34, 16400, 600)])
def test_sizes(T, Na, Nb):
    p = gpu()
    say(f"[ordered] {T} x {Na} x {Nb}")
    r = np.random.default_rng(Na + Nb)
    A, B = _cloth(r, T, Na), _cloth(r, T, Nb)
    if T > 4:  # the first and the last frames
        g = {k: host(v) for k, v in p.chamfer_fwd(dev(A), dev(B)).items()}
        for t in (0, T - 1):
            for q, c, side in ((A, B, "a"), (B, A, "b")):
                idx, d32, _ = oracle.nearest(q[t], c[t])
                assert np.array_equal(g["idx_" + side][t], idx)
                assert np.array_equal(g["dist_" + side][t].view(np.uint32), d32.view(np.uint32))
    else:
        _check(p, A, B)
        _check(p, A, B, two=False)


def _clouds(kind, r, n):
    A, B = _cloth(r, 1, n), _cloth(r, 1, n + 37)
    if kind == "padded":        # a third of both clouds is one repeated point, as in padded scans
        A[0, r.choice(n, n // 3, replace=False)] = 0
        B[0, r.choice(n, n // 3, replace=False)] = 0
    elif kind == "identical":   # both clouds one repeated point each
        A[0], B[0] = A[0, 0], B[0, 0]
    elif kind == "lattice":     # eight equidistant neighbours, every point twice
        x = np.arange(16, dtype=np.float32) / 16
        G = np.stack(np.meshgrid(x, x, x, indexing="ij"), -1).reshape(1, -1, 3)
        A = np.concatenate([G, G], 1)[:, r.permutation(2 * G.shape[1])]
        B = (A[:, ::2] + np.float32(1 / 32)).copy()
    elif kind == "stray":       # a few points far away, and one far beyond
        A[0, ::997] = r.normal(0, 1e4, A[0, ::997].shape)
        B[0, 5] = 1e20
        B[0, 6] = -3e17
    elif kind == "far":         # clouds well apart
        B += np.float32([3, -40, 7])
    elif kind == "line":        # no extent on two axes
        A[..., 1:] = 0.25
        B[..., 1:] = 0.25
    elif kind == "tiny":        # distances that underflow to zero, all tied
        A *= np.float32(1e-24)
        B *= np.float32(1e-24)
    elif kind == "sphere":      # no box rules anything out for points at the centre
        u = r.normal(size=(1, n, 3))
        A = (u / np.linalg.norm(u, axis=2, keepdims=True)).astype(np.float32)
        B = (r.normal(size=(1, n, 3)) * 1e-3).astype(np.float32)
    return A, B


@pytest.mark.parametrize("n", [3000, 17000])
@pytest.mark.parametrize("kind", ["padded", "identical", "lattice", "stray", "far", "line", "tiny",
                                  "sphere"])
def test_clouds(kind, n):
    p = gpu()
    say(f"[ordered] {kind} {n}")
    A, B = _clouds(kind, np.random.default_rng(n), n)
    _check(p, A, B)


@pytest.mark.parametrize("T,n", [(1, 1500), (60, 1500), (2, 20000)])
def test_not_finite(T, n):
    """Points that are NaN or whose squares overflow, a frame of NaN queries and a frame of NaN
    targets: what the exhaustive search gives, a NaN distance never winning and, where none is
    finite, the first of the first 64 targets at an infinite distance or target 0."""
    p = gpu()
    say(f"[ordered] not finite {T} x {n}")
    r = np.random.default_rng(n + T)
    A, B = _cloth(r, T, n), _cloth(r, T, n)
    for X in (A, B):
        X[0, ::50, 1] = np.nan
        X[0, 7::90] = 4e30
        X[0, 11, 0] = np.inf
        X[0, 12, 2] = -np.inf
    if T > 1:
        A[T - 1] = np.nan
        B[T // 2, :, 0] = 5e30
    g = {k: host(v) for k, v in p.chamfer_fwd(dev(A), dev(B)).items()}

    def exhaustive(Q, P):
        with np.errstate(all="ignore"):
            best = np.full(len(Q), np.inf, np.float32)
            for i in range(0, len(Q), 200):
                d = Q[i:i + 200, None] - P[None]  # float32 throughout; fma in double, rounded once
                s = (d[..., 0] * d[..., 0]).astype(np.float64)
                for k in (1, 2):
                    x = d[..., k].astype(np.float64)
                    s = (x * x + s).astype(np.float32).astype(np.float64)
                s = s.astype(np.float32)
                s[np.isnan(s)] = np.inf
                best[i:i + 200] = s.min(1)
        return best

    for t in (0, T - 1, T // 2):
        for Q, P, side in ((A, B, "a"), (B, A, "b")):
            some = slice(t % 3, None, 3 if n < 5000 else 25)
            Qs, got, gd = Q[t][some], g["idx_" + side][t][some], g["dist_" + side][t][some]
            best = exhaustive(Qs, P[t])
            fin = np.isfinite(best)
            assert np.array_equal(np.isfinite(gd), fin), (t, side)
            assert np.allclose(gd[fin], best[fin], rtol=1e-6, atol=0)
            assert got.min() >= 0 and got.max() < n
            with np.errstate(all="ignore"):
                dg = Qs.astype(np.float64) - P[t][got].astype(np.float64)
                assert np.allclose((dg[fin] ** 2).sum(1), best[fin], rtol=1e-6, atol=0)
                for q in np.nonzero(~fin)[0][:200]:
                    d = Qs[q][None] - P[t][:64]
                    s = (d * d).sum(1)
                    inf = np.nonzero(np.isposinf(s))[0]
                    assert got[q] == (inf[0] if len(inf) else 0), (t, side, q)


def test_budget_without_room_for_the_ordered_clouds():
    """A budget that holds the exact search's scratch but not the ordered clouds: the direct call and
    the served request still run, with the same results."""
    p = gpu()
    from paper_2204_03139_amd.serving import Server
    say("[ordered] short budget")
    r = np.random.default_rng(3)
    A, B = _cloth(r, 40, 4096), _cloth(r, 40, 4096)
    ref = {k: host(v) for k, v in p.chamfer_fwd(dev(A), dev(B)).items()}
    ctx = p.Context(0, hbm_budget_bytes=6 << 20)
    g = {k: host(v) for k, v in p.chamfer_fwd(dev(A), dev(B), ctx=ctx).items()}
    assert ctx.memory_held()[0] <= 6 << 20
    ctx.close()
    for k, v in ref.items():
        assert np.array_equal(g[k].view(np.uint8), v.view(np.uint8)), k
    from workloads import gen
    verts, faces = gen.trajectory(6, 20, 5)
    obs = _cloth(r, 20, 4096)
    need = Server.footprint(verts, faces, obs, 4096, precision=0, want_grad=False)
    res = []
    for budget in (1 << 30, need + (1 << 20)):  # the loop's own descriptors take more than 1 MiB
        srv = Server(hbm_budget_bytes=budget)
        st, loss, _, _ = srv.wait(srv.submit(verts, faces, obs, 4096, 5, 0, want_grad=False))
        assert st == 0
        res.append(loss)
        srv.close()
    assert np.array_equal(res[0], res[1])
