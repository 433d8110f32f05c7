"""The face choice of the sampler (Sec. III-B, Eq. 3) where its search tree, its blocks of faces and its
shares of points begin and end: faces, points and weights bit for bit those of the oracle."""
import numpy as np
import pytest

import oracle
from workloads import gen

from gpu_helpers import dev, gpu, host, say, torch

pytestmark = pytest.mark.gpu


def _strip(T, F, V, seed):
    """F faces over V vertices: uneven triangles, every ninth of zero area."""
    r = np.random.default_rng(seed)
    verts = r.standard_normal((T, V, 3)).astype(np.float32)
    faces = np.stack([r.permutation(V)[:3] if V < 64 else r.integers(0, V, 3) for _ in range(F)])
    faces[8::9, 1] = faces[8::9, 2]
    return verts, faces.astype(np.int32)


def _even(F):
    """F equal triangles of area 2^-7: the sums are multiples of one step."""
    v = np.zeros((1, F + 2, 3), np.float32)
    v[0, :, 0] = np.arange(F + 2) // 2 * 0.125
    v[0, 1::2, 1] = 0.125
    k = np.arange(F)
    return v, np.stack([k, k + 1, k + 2], 1).astype(np.int32)


def _words(T, N, seed):
    w = np.random.default_rng(seed).integers(0, 2**32, (T, N, 4), dtype=np.uint64).astype(np.uint32)
    w[:, 0, :2] = 0                # the first face
    w[:, N // 2, :2] = 2**32 - 1   # the last
    return w


def _same(got, exp):
    for g, e in zip(got, exp):
        g, e = np.ascontiguousarray(host(g)), np.ascontiguousarray(e)
        assert np.array_equal(g.view(np.uint32), e.view(np.uint32))


@pytest.mark.parametrize("T,F,V,N", [
    (1, 1, 3, 1), (2, 2, 4, 511), (3, 3, 5, 513), (1, 7, 6, 4097), (1, 4095, 900, 700),
    (2, 4096, 901, 5000), (1, 8191, 5000, 2048), (1, 16385, 20000, 1025),
    # enough points for the wide kernel: shares of one frame, of several, and of a part of two
    (1, 1, 3, 1 << 19), (64, 2047, 1500, 8192), (53, 4095, 700, 10007), (2, 8192, 12800, 1 << 18),
    (64, 40, 12801, 8192),  # corners of one vertex too many for it
])
@pytest.mark.parametrize("words", [True, False])
def test_faces_points_and_weights(T, F, V, N, words):
    p = gpu()
    say(f"[sampler] {T} x {F} faces, {N} points, words {words}")
    verts, faces = _strip(T, F, V, F + N)
    if F == 1:
        verts[:] = np.float32([[0, 0, 0], [1, 0, 0], [0, 1, 0]])
    w = _words(T, N, F) if words else None
    g = p.sample_surface(dev(verts), dev(faces), N, seed=9,
                         uniforms=dev(w.view(np.int32)) if words else None)
    _same(g, oracle.sample_surface(verts, faces, N, words=w, seed=9))


@pytest.mark.parametrize("F,N", [(64, 300), (4096, 9000), (16384, 16384), (8192, 1 << 19)])
def test_draws_that_equal_a_sum(F, N):
    """r S = C_k exactly: the face is k + 1, never k."""
    p = gpu()
    verts, faces = _even(F)
    w = _words(1, N, 3)
    k = np.random.default_rng(F).integers(0, F, N)
    w[0, :, 0] = 0
    w[0, :, 1] = k << (32 - F.bit_length() + 1)
    g = p.sample_surface(dev(verts), dev(faces), N, uniforms=dev(w.view(np.int32)))
    assert np.array_equal(host(g[1])[0], k)
    _same(g, oracle.sample_surface(verts, faces, N, words=w))


@pytest.mark.parametrize("N", [300, 8192])
def test_degenerate_frame_between_others(N):
    """One frame without area: its points are NaN, its faces -1, and the others are as ever."""
    p = gpu()
    T = 64
    verts, faces = gen.trajectory(5, T, 9)
    verts[17] = 0.0
    w = _words(T, N, 5)
    ctx = p.Context(0)
    g = [host(x) for x in p.sample_surface(dev(verts), dev(faces), N,
                                           uniforms=dev(w.view(np.int32)), ctx=ctx)]
    with pytest.raises(p.DCError):
        ctx.sync()
    ctx.close()
    assert np.isnan(g[0][17]).all() and (g[1][17] == -1).all() and (g[2][17] == 0).all()
    good = np.arange(T) != 17
    _same([torch.from_numpy(x[good]) for x in g],
          oracle.sample_surface(verts[good], faces, N, words=w[good]))
