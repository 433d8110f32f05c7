"""Clouds of hundreds of thousands to millions of points (Sec. III-A, Eq. 1-2): many parts, cells of many points,
one or two frames.  The ordered search equals the search that evaluates every pair, bit for bit."""
import pytest

from gpu_helpers import gpu, say, torch

pytestmark = pytest.mark.gpu


def _cloud(kind, n, g):
    def randn(*s):
        return torch.randn(s, generator=g, device="cuda")
    if kind == "sphere":
        u = randn(n, 3)
        return u / u.norm(dim=1, keepdim=True)
    if kind == "point":
        return randn(n, 3) * 1e-3
    xy = torch.rand((n, 2), generator=g, device="cuda") - .5
    X = torch.cat([xy, .05 * torch.sin(12 * xy[:, :1]) + .005 * randn(n, 1)], 1)
    if kind == "clumps":
        X += 5 * torch.randint(0, 3, (n, 3), generator=g, device="cuda")
    elif kind == "twice":       # every point a second time, elsewhere in the cloud
        X[n // 2:2 * (n // 2)] = X[:n // 2].clone()
    return X


@pytest.mark.parametrize("a,b,T,n,m", [("sheet", "sheet", 1, 2_100_001, 1_000_003), ("clumps", "clumps", 2, 262_144, 300_001),
                                       ("point", "sphere", 1, 150_000, 262_145), ("twice", "twice", 1, 400_000, 400_000),
                                       ("clumps", "clumps", 1, 1_048_576, 700_000)])
def test_large(a, b, T, n, m):
    p = gpu()
    say(f"[large] {a} {b} {T} x {n} x {m}")
    g = torch.Generator(device="cuda")
    g.manual_seed(n)
    A = torch.stack([_cloud(a, n, g) for _ in range(T)]).contiguous()
    B = torch.stack([_cloud(b, m, g) for _ in range(T)]).contiguous()
    ctx = p.Context(0)
    got = p.chamfer_fwd(A, B, ctx=ctx)
    ctx.debug_search(3)
    every = p.chamfer_fwd(A, B, ctx=ctx)
    torch.cuda.synchronize()
    for k in every:
        assert torch.equal(got[k], every[k]), k
    ctx.close()


def test_most_frames():
    """65,535 frames, the most a call takes, of clouds that are ordered."""
    p = gpu()
    say("[large] 65535 frames of 40 x 33")
    g = torch.Generator(device="cuda")
    g.manual_seed(1)
    A, B = (torch.rand((65535, k, 3), generator=g, device="cuda") for k in (40, 33))
    ctx = p.Context(0)
    out = []
    for search in (1, 3):
        ctx.debug_search(search)
        out.append(p.chamfer_fwd(A, B, ctx=ctx))
    torch.cuda.synchronize()
    for k in out[0]:
        assert torch.equal(out[0][k], out[1][k]), k
    ctx.close()
