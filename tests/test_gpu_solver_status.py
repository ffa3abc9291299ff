"""The status that a time step's solves publish to the host: converged steps report
true residuals and repeat bit for bit, a solve out of iterations or with a
non-finite value is an error of the step that leaves the state, and the solver
works on afterwards; for the three viscous solves (Jacobi sweeps, BiCGSTAB, mixed
precision) in front of the flexible GMRES."""
import pytest

import rbf_inputs as ri
from tests.helpers import to_dev, gpu_cavity_ops

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("re,dt,precision", [(1e4, 2e-4, "fp64"), (50.0, 5e-3, "fp64"),
                                             (1e4, 2e-4, "mixed")])
def test_status(gpu, re, dt, precision):
    import torch
    import paper_2206_06495_amd as P
    nd = ri.hex_cavity_nodes(14, 0.3, 1)
    grid, ops = gpu_cavity_ops(nd, gpu)
    u_bc, v_bc = (to_dev(b, gpu) for b in ri.cavity_bc(nd.v_tag))

    def solver(**kw):
        return P.Solver(grid, ops, u_bc, v_bc, re, dt, precision=precision, **kw)

    S = solver()
    runs = []
    for _ in range(2):
        st = S.new_state(u_bc, v_bc)
        stats = S.step(st, 4)
        # BiCGSTAB stops on its recursive residual: 1e-13 and the rounding of some
        # ten updates, each of a few u times the condition number (below 100)
        for h in (stats.last_helmholtz_u, stats.last_helmholtz_v):
            assert h.converged and 0.0 < h.rel_residual <= 1e-11
        p = stats.last_poisson
        assert p.converged and p.final_flag == 1 and p.restarts >= 1 and 0.0 < p.rel_residual <= 1e-12
        assert stats.poisson_iters >= p.iterations > 0
        runs.append(st)
    for key in ("u", "v", "p", "p_tilde"):
        assert torch.equal(runs[0][key], runs[1][key]), key
    for kw in ({"maxit_h": 1}, {"maxit_p": 1}):
        B = solver(**kw)
        st = B.new_state(u_bc, v_bc)
        with pytest.raises(P.RbfError) as err:
            B.step(st, 1)
        assert err.value.status == -3 and st["step"] == 0 and torch.equal(st["u"], u_bc), kw
        B.close()
    bad = S.new_state(u_bc, v_bc)
    bad["u"][nd.v_tag.shape[0] // 2] = float("nan")
    with pytest.raises(P.RbfError) as err:
        S.step(bad, 1)
    assert err.value.status == -6 and bad["step"] == 0
    st = S.new_state(u_bc, v_bc)
    S.step(st, 4)
    assert torch.equal(st["u"], runs[0]["u"])
    S.close()
