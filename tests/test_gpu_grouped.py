"""The backward's sums over small segments (Chamfer backward, Sec. III-A; sampling backward, Eq. 4):
the sums of every key in double against numpy's, and bit for bit the same on every run, at the edges of a
workgroup's range, of its list (keys with more items than it holds, ranges that take several rounds),
of the teams of lanes, of the two workgroup sizes and of the path that sorts instead."""
import numpy as np
import pytest

from gpu_helpers import dev, gpu, host, say, torch

pytestmark = pytest.mark.gpu


def _keys(kind, r, T, n, K):
    if kind == "uniform":
        k = r.integers(0, K, (T, n))
    elif kind == "one":          # every item the same key
        k = np.full((T, n), K // 2)
    elif kind == "skewed":       # half the items in a few neighbouring keys, some out of range
        k = np.where(r.random((T, n)) < .5, r.integers(0, max(1, K // 100), (T, n)),
                     r.integers(0, K, (T, n)))
        k[:, ::17] = -1
        k[:, 5::31] = K
    elif kind == "sorted":
        k = np.sort(r.integers(0, K, (T, n)), 1)
    return k.astype(np.int32)


# Each output is a sum of doubles rounded once (chamfer), or sums rounded once and summed again
# (vertices): with u = 2^-24 at most 2 u of the sum of the terms' magnitudes, and a little for the
# double sums themselves.
BOUND = 2.1 * 2.0 ** -24


@pytest.mark.parametrize("kind", ["uniform", "one", "skewed", "sorted"])
@pytest.mark.parametrize("T,Na,Nb", [(1, 1, 1), (3, 63, 2047), (2, 2048, 2049), (1, 7, 5000),
                                     (40, 300, 9000), (1, 32768, 32769), (2, 40000, 700),
                                     (1, 131072, 131073)])
def test_chamfer_backward(kind, T, Na, Nb):
    p = gpu()
    say(f"[grouped] chamfer {kind} {T} x {Na} x {Nb}")
    r = np.random.default_rng(Na * 7 + Nb)
    A = r.uniform(-.5, .5, (T, Na, 3)).astype(np.float32)
    B = r.uniform(-.5, .5, (T, Nb, 3)).astype(np.float32)
    ia, ib = _keys(kind, r, T, Na, Nb), _keys(kind, r, T, Nb, Na)
    g = r.uniform(.5, 2, T)
    out = [p.chamfer_bwd(dev(g), dev(A), dev(B), dev(ia), dev(ib), want_b=True) for _ in range(2)]
    ga, gb = (host(x) for x in out[0])
    for x, y in zip(out[0], out[1]):
        assert np.array_equal(host(x).view(np.uint32), host(y).view(np.uint32))
    al, be = 1.0 / Na, 1.0 / Nb
    for t in range(T):
        ea, eb = np.zeros((Na, 3)), np.zeros((Nb, 3))
        ma, mb = np.zeros((Na, 3)), np.zeros((Nb, 3))
        a, b = A[t].astype(np.float64), B[t].astype(np.float64)
        for (q, c, nn, w, eq, ec, mq, mc) in ((a, b, ia[t], al, ea, eb, ma, mb),
                                              (b, a, ib[t], be, eb, ea, mb, ma)):
            ok = np.nonzero((nn >= 0) & (nn < len(c)))[0]
            d = 2 * w * g[t] * (q[ok] - c[nn[ok]])
            eq[ok] += d
            mq[ok] += np.abs(d)
            np.subtract.at(ec, nn[ok], d)
            np.add.at(mc, nn[ok], np.abs(d))
        assert np.all(np.abs(ga[t] - ea) <= BOUND * ma + 1e-30), t
        assert np.all(np.abs(gb[t] - eb) <= BOUND * mb + 1e-30), t


@pytest.mark.parametrize("kind", ["uniform", "one", "skewed"])
@pytest.mark.parametrize("T,V,F,N", [(1, 3, 1, 5000), (65, 40, 72, 3500), (2, 3000, 5900, 2047),
                                     (2, 50, 5000, 32769), (1, 30000, 43691, 131072),
                                     (1, 500, 900, 131073)])
def test_sampling_backward(kind, T, V, F, N):
    p = gpu()
    say(f"[grouped] sampling {kind} {T} x {V} x {F} x {N}")
    r = np.random.default_rng(V + F + N)
    faces = r.integers(0, V, (F, 3)).astype(np.int32)
    fi = _keys(kind, r, T, N, F)
    fi[fi == F] = -1
    g = r.normal(size=(T, N, 3)).astype(np.float32)
    w = r.uniform(0, 1, (T, N, 3)).astype(np.float32)
    out = [p.sample_surface_bwd(dev(g), dev(faces), dev(fi), dev(w), V) for _ in range(2)]
    assert torch.equal(out[0], out[1])
    gv = host(out[0])
    for t in range(0, T, 16):
        e, m = np.zeros((V, 3)), np.zeros((V, 3))
        ok = fi[t] >= 0
        for c in range(3):
            d = w[t, ok, c, None].astype(np.float64) * g[t, ok].astype(np.float64)
            np.add.at(e, faces[fi[t, ok], c], d)
            np.add.at(m, faces[fi[t, ok], c], np.abs(d))
        assert np.all(np.abs(gv[t] - e) <= BOUND * m + 1e-30), t
