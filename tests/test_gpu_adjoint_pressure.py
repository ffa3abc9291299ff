"""The adjoint step's transposed pressure solve by preconditioned flexible
GMRES: every kind of solver that builds its structures its own way (shared with
the forward solve, beside the lattice preconditioner, beside FP32 structures,
without a preconditioner), and the smallest set, which keeps BiCGSTAB."""
import numpy as np
import pytest

import rbf_inputs as ri
from oracle import adjoint as oadj, cavity as ocav
from tests.helpers import to_dev, gpu_cavity_ops

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kind,K,kw", [(2, 14, {}), (0, 12, {}), (2, 12, {"precision": "mixed"}),
                                       (0, 12, {"precision": "mixed"}), (0, 10, {"precond": "none"}),
                                       (0, 6, {})])
def test_gradient_against_the_oracle(gpu, kind, K, kw):
    """Five steps, rtol_p = 1e-13: within 1e-8 of the largest component, as the
    rollout tests (the solves' tolerance times the systems' conditioning)."""
    import torch
    import paper_2206_06495_amd as P
    print(kind, K, kw, flush=True)
    nd = ri.cavity_nodes(K, 0.3, 4) if kind == 0 else ri.hex_cavity_nodes(K, 0.3, 4)
    grid, ops = gpu_cavity_ops(nd, gpu)
    lid = nd.v_tag == ri.TAG_LID
    modes = np.sin(np.pi * np.outer(np.arange(1, 9), nd.xv[0])) * lid
    coef = np.array([1.0, 0.0, -0.3, 0.1, 0.0, 0.0, 0.2, 0.0])
    dt, nu, nsteps = 2e-3, 1e-2, 5
    R = P.LidRollout(grid, ops, to_dev(modes, gpu), dt, nsteps, every=3, rtol_p=1e-13, **kw)
    nu_t = torch.tensor(nu, dtype=torch.float64, requires_grad=True)
    c_t = torch.tensor(coef, dtype=torch.float64, requires_grad=True)
    R(nu_t, c_t).backward()
    orc = ocav.CavityOracle(nd, coef @ modes, np.zeros(nd.n_v), 1.0 / nu, dt, dense=True)
    _, nub, ubc_b, _, _ = oadj.rollout_gradient(orc, orc.initial_state(), nsteps)
    go = modes @ ubc_b
    assert abs(float(nu_t.grad) - nub) <= 1e-8 * abs(nub)
    assert np.max(np.abs(c_t.grad.numpy() - go)) <= 1e-8 * np.max(np.abs(go))
