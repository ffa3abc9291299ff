"""kNN on uneven source sets, where the search raises its window, skips or repeats a
pass or keeps only the lowest indices of a distance: crowded cells beside empty
ones, a far outlier, coincident sources beyond the list's length, queries outside the
box on every side.  Against brute force, bit for bit."""
import numpy as np
import pytest

from oracle import knn as oknn
from tests.helpers import to_dev

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def P(gpu):
    import paper_2206_06495_amd as P
    return P


def _sources(name):
    r = np.random.default_rng(11)
    u = r.random((2, 1400))
    return {"heavy tails": lambda: r.standard_normal((2, 1500)) ** 3,
            "outlier": lambda: np.concatenate([u, [[1e4], [1e4]]], axis=1),
            "crowded corner": lambda: np.concatenate([u * 1e-3, u], axis=1),
            "clusters": lambda: r.random((2, 9))[:, r.integers(0, 9, 1500)] + 1e-3 * r.standard_normal((2, 1500)),
            "layer": lambda: np.stack([u[0], np.exp(-8 * u[1])]),
            "copies": lambda: np.repeat(r.random((2, 20)), 80, axis=1)[:, r.permutation(1600)],
            "rings": lambda: np.stack([np.cos(np.arange(1200) * np.pi / 2), np.sin(np.arange(1200) * np.pi / 2)])
                             * np.repeat(np.arange(1.0, 5.0), 300),
            }[name]()


@pytest.mark.parametrize("name", ["heavy tails", "outlier", "crowded corner", "clusters", "layer", "copies",
                                  "rings"])
@pytest.mark.parametrize("k", [1, 5, 16, 28, 32, 48, 49, 64])
def test_against_brute_force(P, gpu, name, k):
    print(name, k, flush=True)
    xs = _sources(name)
    lo, hi = xs.min(axis=1, keepdims=True), xs.max(axis=1, keepdims=True)
    some = xs[:, ::41]
    parts = [xs[:, ::13], 0.5 * (some + np.roll(some, 7, axis=1))]
    for a in (-1, 0, 1):
        for b in (-1, 0, 1):
            for far in (0.3, 12.0):
                parts.append(some + far * np.array([[a], [b]]) * (hi - lo))
    xq = np.concatenate(parts, axis=1)
    idx = P.knn(to_dev(xq, gpu), to_dev(xs, gpu), k).cpu().numpy()
    assert np.array_equal(idx, oknn.knn_bruteforce(xq, xs, k))
