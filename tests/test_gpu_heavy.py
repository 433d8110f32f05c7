"""The backward's sums where a few neighbouring keys hold most items (Chamfer backward, Sec. III-A; sampling
backward, Eq. 4): keys at both sides of the line between ranked and workgroup-wide sums, several of those in a
row, rounds of few long keys, ones that overflow a workgroup's list, between ordinary keys and at the ends of a range."""
import math

import numpy as np
import pytest

import test_gpu_grouped as grouped

pytestmark = pytest.mark.gpu


def _keys(kind, r, T, n, K):
    line = math.isqrt(12 * n)  # the most items of an ordinary key
    runs = dict(line=[line, line + 1, line - 1, line + 1, line + 1],
                runs=[5, 3 * line, 7, 9, 2 * line, 2 * line, 1],
                over=[line, 4097, 3, 2049, 2 * line, 2048],
                round=[line // 3] * 9,
                # rounds of few long keys, a list's fill of them and one item more, with ordinary ones between
                long=[line // 3] * 30 + [2, 5] + [256] * 17 + [128] * 33 + [257, 129, line // 2] * 8)[kind]
    k = np.empty((T, n), np.int32)
    for t in range(T):
        first = int(r.integers(0, max(1, K - len(runs)))) if t else 0  # at the first key's range, anywhere
        own = np.concatenate([np.full(m, min(first + j, K - 1)) for j, m in enumerate(runs)])[:n]
        k[t] = np.concatenate([own, r.integers(0, K, n - len(own))])[r.permutation(n)]
    return k


@pytest.mark.parametrize("kind", ["line", "runs", "over", "round", "long"])
@pytest.mark.parametrize("T,Na,Nb", [(3, 700, 9000), (2, 30000, 20011), (1, 65536, 49153), (1, 300, 131072)])
def test_chamfer_backward(monkeypatch, kind, T, Na, Nb):
    monkeypatch.setattr(grouped, "_keys", _keys)
    grouped.test_chamfer_backward(kind, T, Na, Nb)


@pytest.mark.parametrize("kind", ["line", "runs", "over", "round", "long"])
@pytest.mark.parametrize("T,V,F,N", [(17, 400, 900, 8192), (1, 10000, 19602, 65536), (2, 3000, 40, 2500)])
def test_sampling_backward(monkeypatch, kind, T, V, F, N):
    monkeypatch.setattr(grouped, "_keys", _keys)
    grouped.test_sampling_backward(kind, T, V, F, N)
