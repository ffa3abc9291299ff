"""The windowed kNN search where its first window, its list or its arithmetic
runs out: stencil sizes around the compiled chain lengths, clustered and
collinear sources, coincident sources, far queries, coordinates whose squares
leave the range of doubles.  Against brute force, bit for bit."""
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
    r = np.random.default_rng(7)
    return {"uniform": lambda: r.random((2, 1501)),
            "clustered": lambda: r.standard_normal((2, 1500)) ** 3,
            "line": lambda: np.stack([r.random(700), np.zeros(700)]),
            "coincident": lambda: np.round(r.random((2, 2000)) * 8) / 8,
            "one point": lambda: np.full((2, 90), 0.25),
            "lattice": lambda: np.stack([g.ravel() for g in np.meshgrid(np.arange(30.0), np.arange(30.0))]),
            "huge": lambda: r.random((2, 300)) * 1e300,
            "tiny": lambda: r.random((2, 300)) * 1e-300}[name]()


@pytest.mark.parametrize("name", ["uniform", "clustered", "line", "coincident", "one point", "lattice",
                                  "huge", "tiny"])
@pytest.mark.parametrize("k", [1, 16, 17, 28, 29, 33, 49, 64])
def test_against_brute_force(P, gpu, name, k):
    print(name, k, flush=True)
    xs = _sources(name)
    span = np.abs(xs).max()
    xq = np.concatenate([xs[:, ::9], xs[:, ::31] * 1.5 - 0.2 * span, [[30 * span], [-7 * span]]], axis=1)
    idx = P.knn(to_dev(xq, gpu), to_dev(xs, gpu), k).cpu().numpy()
    with np.errstate(over="ignore"):
        assert np.array_equal(idx, oknn.knn_bruteforce(xq, xs, k))
