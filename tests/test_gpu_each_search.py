"""Every nearest-neighbour search by itself (Sec. III-A, Eq. 1-2), wherever the library would choose another one:
over ordered clouds, the bf16 screen with its exact re-evaluation, and every pair in single precision.  They are
compared with each other bit for bit, and each runs the tests that hold its edges: column merges and their ties,
heavy lists, coordinate scales, both directions in one pass, requests batched with others."""
import numpy as np
import pytest

import oracle
import test_gpu_ordered as ordered
import test_gpu_parity as parity
import test_gpu_serving as serving
import test_gpu_sweep as sweep

from gpu_helpers import dev, gpu, host, say

pytestmark = pytest.mark.gpu

ORDERED, SCREEN, EXACT = 1, 2, 3
NAMES = {ORDERED: "ordered", SCREEN: "screen", EXACT: "exact"}


@pytest.fixture
def force(monkeypatch):
    """Sets the search of the default context and of every context made in the test."""
    p = gpu()
    from paper_2204_03139_amd import _lib
    init = _lib.Context.__init__

    def to(search):
        say(f"[each search] {NAMES[search]}")
        p.default_context().debug_search(search)

        def made(self, *a, **k):
            init(self, *a, **k)
            self.debug_search(search)
        monkeypatch.setattr(_lib.Context, "__init__", made)

    yield to
    p.default_context().debug_search(0)


def _not_finite(r, T, n, m):
    A, B = ordered._cloth(r, T, n), ordered._cloth(r, T, m)
    for X in (A, B):
        k = X.shape[1]
        X[0, r.choice(k, k // 40, replace=False), r.integers(0, 3)] = np.nan
        X[0, r.choice(k, k // 90, replace=False)] = 4e30
        X[0, r.integers(0, k), 0] = np.inf
    A[T - 1] = np.nan
    B[T // 2, :, 0] = 5e30
    return A, B


CLOUDS = {
    "cloth": lambda r, T, n, m: (ordered._cloth(r, T, n), ordered._cloth(r, T, m)),
    "not finite": _not_finite,
    "repeated": lambda r, T, n, m: tuple(np.where(r.random((T, k, 1)) < .4, np.float32(.1), X)
                                         for k, X in ((n, ordered._cloth(r, T, n)), (m, ordered._cloth(r, T, m)))),
    "apart": lambda r, T, n, m: (ordered._cloth(r, T, n), ordered._cloth(r, T, m) + np.float32([30, 0, 4])),
    "sphere": lambda r, T, n, m: tuple(np.stack(x) for x in
                                       zip(*(sweep._frame("ties", r, n, m) for _ in range(T)))),
}


# one small frame, lopsided clouds, slices of the targets, many frames in one pass, more than one part
@pytest.mark.parametrize("T,n,m", [(3, 1, 5), (3, 700, 64), (1, 8193, 130), (3, 900, 21000), (270, 520, 300),
                                   (4, 17000, 3000)])
@pytest.mark.parametrize("kind", list(CLOUDS))
def test_same_results(kind, T, n, m):
    p = gpu()
    say(f"[each search] {kind} {T} x {n} x {m}")
    A, B = CLOUDS[kind](np.random.default_rng(n + m), T, n, m)
    ctx = p.Context(0)
    for two in (True, False):
        kw = dict(ctx=ctx) if two else dict(ctx=ctx, reduction=1, b_side=False)
        got = {}
        for search in NAMES:
            ctx.debug_search(search)
            got[search] = {k: host(v) for k, v in p.chamfer_fwd(dev(A), dev(B), **kw).items() if v is not None}
        exact = got[EXACT]
        for k, v in exact.items():
            assert np.array_equal(v.view(np.uint8), got[ORDERED][k].view(np.uint8)), ("ordered", two, k)
        # (the screen may give NaN for a query without a finite distance, and any index)
        for side in "ab"[:2 if two else 1]:
            fin = np.isfinite(exact["dist_" + side])
            assert np.array_equal(fin, np.isfinite(got[SCREEN]["dist_" + side])), ("screen", two, side)
            for k in ("dist_" + side, "idx_" + side):
                same = exact[k].view(np.uint32) == got[SCREEN][k].view(np.uint32)
                assert same[fin].all(), ("screen", two, k)
        if kind != "not finite":
            for t in (0, T - 1):
                idx, d32, _ = oracle.nearest(A[t], B[t])
                assert np.array_equal(got[EXACT]["idx_a"][t], idx)
                assert np.array_equal(got[EXACT]["dist_a"][t].view(np.uint32), d32.view(np.uint32))
    ctx.close()


@pytest.mark.parametrize("search", list(NAMES))
@pytest.mark.parametrize("case", list(parity.CHAMFER_CASES))
def test_parity(force, search, case):
    force(search)
    parity.test_chamfer_parity(case, search % 2)


@pytest.mark.parametrize("search", list(NAMES))
def test_ties(force, search):
    force(search)
    parity.test_chamfer_ties_and_identity(0)


@pytest.mark.parametrize("search", [SCREEN, EXACT])
@pytest.mark.parametrize("case", list(parity.COLUMN_MERGE_CASES))
def test_column_merge(force, search, case):
    force(search)
    parity.test_column_merge_ties_and_list_overflow(case, 0)


@pytest.mark.parametrize("search", [SCREEN, EXACT])
@pytest.mark.parametrize("scale", [1e-12, 1e-6, 1e6, 1e12])
def test_scales(force, search, scale):
    force(search)
    parity.test_coordinate_scales(scale, 0)


@pytest.mark.parametrize("n", [6000, 20000])
def test_heavy_lists(force, n):
    force(SCREEN)
    parity.test_short_heavy_lists(n)


@pytest.mark.parametrize("search", [SCREEN, EXACT])
@pytest.mark.parametrize("shape", [(300, 1000, 777), (260, 2300, 5000), (1100, 2048, 300)])
def test_one_pass(force, search, shape):
    force(search)
    parity.test_one_pass_both_directions(shape)


def test_screen_statistics(force):
    force(SCREEN)
    parity.test_screen_candidates_are_few()


@pytest.mark.parametrize("search", list(NAMES))
def test_requests(force, search):
    force(search)
    serving.test_batched_options_match_direct_calls()
