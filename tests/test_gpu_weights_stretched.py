"""Weights of the paper's stencil on node sets squeezed in y, where k_weights_quad takes
some rows and leaves others to the pivoted kernels: none of the rows at 1:4 and 1:16, a
few at 1:32, most at 1:64, all at 1:256 (wavefronts that end early).  Which rows are left
is seen from the bits: with the condition estimate they come from another kernel than
without, while the rows that are not left are the same.  (Which ones exactly cannot be
told beforehand: the ten nodes are chosen in FP32, whose rounding is of the size of the
smallest pivots there.)"""
import ctypes

import numpy as np
import pytest

import rbf_inputs as ri
from oracle import knn as oknn, weights as ow
from tests.helpers import OP_DX, OP_DY, OP_LAP, to_dev

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def P(gpu):
    import paper_2206_06495_amd as P
    return P


def _row_errors(w, ref):
    return np.abs(w - ref).max(axis=0) / np.abs(ref).max(axis=0)


@pytest.mark.parametrize("squeeze,left_rows", [(2, (0, 0)), (4, (0, 0)), (5, (1, 30)), (6, (100, 134)), (8, (134, 134))])
def test_both_kernels_on_stretched_rows(P, gpu, squeeze, left_rows):
    nd = ri.square_nodes(20, 0.3, 1)
    rows = np.arange(0, nd.xv.shape[1], 3)
    idx = oknn.knn(nd.xv[:, rows], nd.xv, 28)
    x = nd.xv * np.array([[1.0], [2.0 ** -squeeze]])
    xq = x[:, rows]
    ops = [OP_DX, OP_DY]
    xt, yt, e = ow.local_coordinates(xq, x, idx)
    # Tolerance: 100 times what numpy's LU leaves after one refinement step with a residual
    # in extended precision (4e-14 at 1:4, 4e-10 at 1:256).
    A, B = ow.augmented_system(xt, yt, 7, 3, ops)
    X, once = np.linalg.solve(A, B), None
    for _ in range(4):
        res = B.astype(np.longdouble) - np.einsum("rij,rjo->rio", A.astype(np.longdouble), X.astype(np.longdouble))
        X = X + np.linalg.solve(A, res.astype(np.float64))
        once = X if once is None else once
    tol = 100 * max(1e-14, float((np.abs(once - X)[:, :28].max(1) / np.abs(X)[:, :28].max(1)).max()))
    assert tol < 1e-6
    ref = np.ldexp(X[:, :28], -e[:, None, None]).transpose(2, 1, 0)
    dq, ds, di = to_dev(xq, gpu), to_dev(x, gpu), to_dev(idx.astype(np.int32), gpu)
    w = P.assemble_weights(dq, ds, di, 7, 3, OP_DX | OP_DY).cpu().numpy()
    wc = P.assemble_weights(dq, ds, di, 7, 3, OP_DX | OP_DY, cond=True)[0].cpu().numpy()
    print("squeeze", squeeze, "tol", tol, flush=True)
    for o in range(2):
        assert _row_errors(w[o], ref[o]).max() <= tol
        assert _row_errors(wc[o], ref[o]).max() <= tol
    left = (w != wc).any(axis=(0, 1))
    assert left_rows[0] <= left.sum() <= left_rows[1]


def test_bad_rows_beside_good_ones_with_the_estimate(P, gpu):
    """As without the estimate: bad rows NaN and the lowest reported, the others with the
    bits and the estimates that they have alone."""
    import torch
    from paper_2206_06495_amd import _lib
    nd = ri.hex_cavity_nodes(14, 0.3, 3)
    ds, xq = to_dev(nd.xv, gpu), nd.xp.copy()
    idx = P.knn(to_dev(xq, gpu), ds, 28)
    mask = OP_DX | OP_DY | OP_LAP
    good, cond = P.assemble_weights(to_dev(xq, gpu), ds, idx, 7, 3, mask, cond=True)
    assert torch.equal(good, P.assemble_weights(to_dev(xq, gpu), ds, idx, 7, 3, mask))
    bad = [10, 21, 33]
    idx[3, bad[0]] = nd.n_v
    idx[5, bad[1]] = idx[4, bad[1]]
    xq[0, bad[2]] = np.nan
    dq = to_dev(xq, gpu)
    w, c, low = torch.empty_like(good), torch.empty_like(cond), ctypes.c_int64(-7)
    p = lambda t: ctypes.c_void_p(t.data_ptr())  # noqa: E731
    rc = _lib.lib.rbf_assemble_weights(p(dq), xq.shape[1], p(ds), nd.n_v, p(idx), 28, 7, 3, mask, p(w), p(c),
                                       ctypes.byref(low), None)
    torch.cuda.synchronize()
    assert rc == _lib.RBF_E_SINGULAR and low.value == bad[0]
    rest = np.setdiff1d(np.arange(xq.shape[1]), bad)
    assert bool(torch.isnan(w[:, :, bad]).all())
    assert torch.equal(w[:, :, rest], good[:, :, rest])
    assert torch.equal(c[rest], cond[rest])
