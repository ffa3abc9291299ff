"""The four-systems-per-wavefront weight kernel (28 nodes, r^7, cubics) at the
edges of its range: numbers of rows around its groups of four, each number of
operators, and rows that it leaves to the pivoted kernel."""
import numpy as np
import pytest

import rbf_inputs as ri
from oracle import weights as ow
from tests.helpers import OP_ID, OP_DX, OP_DY, OP_LAP, row_rel_err, to_dev

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def P(gpu):
    import paper_2206_06495_amd as P
    return P


@pytest.mark.parametrize("nq", [1, 2, 3, 4, 5, 31, 65])
@pytest.mark.parametrize("mask", [OP_ID, OP_DX | OP_LAP, OP_ID | OP_DX | OP_DY, OP_DX | OP_DY | OP_LAP])
def test_row_counts_and_operators(P, gpu, nq, mask):
    nd = ri.hex_cavity_nodes(12, 0.3, 6)
    xq = nd.xp[:, :nq]
    dq, ds = to_dev(xq, gpu), to_dev(nd.xv, gpu)
    idx = P.knn(dq, ds, 28)
    w = P.assemble_weights(dq, ds, idx, 7, 3, mask).cpu().numpy()
    ops = [c for c in (OP_ID, OP_DX, OP_DY, OP_LAP) if mask & c]
    ref = ow.stencil_weights(xq, nd.xv, idx.cpu().numpy(), 7, 3, ops)
    for o in range(len(ops)):
        assert row_rel_err(w[o], ref[o]) <= 1e-12


def test_stretched_stencils_take_the_pivoted_kernel(P, gpu):
    """Nodes squeezed by 2^-8 in y: the monomial y^3 is below 2^-20, so the
    rows are left to k_weights_pair.  Tolerance: 100 eps times the squared
    condition number of the local systems times eps (one refinement step
    leaves (cond eps)^2), at least 1e-12."""
    nd = ri.square_nodes(14, 0.3, 2)
    x = nd.xv * np.array([[1.0], [2.0 ** -8]])
    rows = np.arange(0, x.shape[1], 7)
    d = to_dev(nd.xv, gpu)
    idx = P.knn(to_dev(nd.xv[:, rows], gpu), d, 28)
    dq, ds = to_dev(x[:, rows], gpu), to_dev(x, gpu)
    w = P.assemble_weights(dq, ds, idx, 7, 3, OP_DX | OP_DY).cpu().numpy()
    _, cond = P.assemble_weights(dq, ds, idx, 7, 3, OP_DX | OP_DY, cond=True)
    tol = max(1e-12, 100 * (float(cond.max()) * 2.0 ** -52) ** 2)
    print("cond", float(cond.max()), "tol", tol, flush=True)
    ref = ow.stencil_weights(x[:, rows], x, idx.cpu().numpy(), 7, 3, [OP_DX, OP_DY])
    for o in range(2):
        assert row_rel_err(w[o], ref[o]) <= tol


def test_left_rows_do_not_touch_their_neighbours(P, gpu):
    """A row with an index out of range, one with coincident stencil nodes and
    one with a non-finite query among good rows: reported and NaN; every
    other row has the bits it has without them."""
    nd = ri.hex_cavity_nodes(14, 0.3, 3)
    ds = to_dev(nd.xv, gpu)
    xq = nd.xp.copy()
    idx = P.knn(to_dev(xq, gpu), ds, 28)
    good = P.assemble_weights(to_dev(xq, gpu), ds, idx, 7, 3, OP_DX | OP_DY | OP_LAP)
    bad = [9, 22, 35]
    idx[3, bad[0]] = nd.n_v
    idx[5, bad[1]] = idx[4, bad[1]]
    xq[0, bad[2]] = np.nan
    import ctypes
    import torch
    from paper_2206_06495_amd import _lib
    dq = to_dev(xq, gpu)
    w = torch.empty_like(good)
    low = ctypes.c_int64(-7)
    p = lambda t: ctypes.c_void_p(t.data_ptr())  # noqa: E731
    rc = _lib.lib.rbf_assemble_weights(p(dq), xq.shape[1], p(ds), nd.n_v, p(idx), 28, 7, 3, 14, p(w),
                                       None, ctypes.byref(low), None)
    torch.cuda.synchronize()
    assert rc == _lib.RBF_E_SINGULAR and low.value == bad[0]
    rest = np.setdiff1d(np.arange(xq.shape[1]), bad)
    assert bool(torch.isnan(w[:, :, bad]).all())
    assert torch.equal(w[:, :, rest], good[:, :, rest])
