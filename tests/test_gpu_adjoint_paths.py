"""Which solvers the adjoint step's transposed systems run on, and the transposed
preconditioner itself: gradients alone cannot tell, since a preconditioner that is
wrong only slows the solve or hands it to the second method."""
import numpy as np
import pytest

import rbf_inputs as ri
from tests.helpers import to_dev, gpu_cavity_ops

pytestmark = pytest.mark.gpu


def _solver(gpu, kind, K, **kw):
    import paper_2206_06495_amd as P
    nd = ri.cavity_nodes(K, 0.3, 4) if kind == 0 else ri.hex_cavity_nodes(K, 0.3, 4)
    grid, ops = gpu_cavity_ops(nd, gpu)
    u_bc, v_bc = ri.cavity_bc(nd.v_tag)
    return nd, P.Solver(grid, ops, to_dev(u_bc, gpu), to_dev(v_bc, gpu), 100.0, 2e-3, **kw), to_dev(u_bc, gpu)


@pytest.mark.parametrize("K", [9, 14, 40, 66, 140])
def test_transposed_preconditioner(gpu, K):
    """<P^-1 a, b> = <a, P^-T b> for every size class of the lattice transforms.  Both
    products' errors grow with the conditioning of the lattice solve, about 0.4 K^2."""
    nd, S, _ = _solver(gpu, 2, K)
    assert S.info()["aux_precond"]
    for seed in (1, 2):
        a, b = ri.random_vector(nd.n_p, seed), ri.random_vector(nd.n_p, seed + 10)
        za = S.apply_precond(to_dev(a, gpu)).cpu().numpy()
        zb = S.apply_precond_t(to_dev(b, gpu)).cpu().numpy()
        scale = np.linalg.norm(za) * np.linalg.norm(b) + np.linalg.norm(a) * np.linalg.norm(zb)
        print(K, seed, abs(za @ b - a @ zb) / scale, flush=True)
        assert abs(za @ b - a @ zb) <= max(1e-12, 4e-16 * K * K) * scale
    S.close()


@pytest.mark.parametrize("kind,K,kw,fast", [(2, 14, {}, True), (2, 40, {}, True), (0, 12, {}, True),
                                            (2, 12, {"precision": "mixed"}, True),
                                            (0, 12, {"precision": "mixed"}, True),
                                            (0, 10, {"precond": "none"}, True), (0, 6, {}, False)])
def test_the_fast_solvers_run(gpu, kind, K, kw, fast):
    """No solve is handed over, the two-component viscous solve runs, and the preconditioned
    pressure solve takes no more than 100 steps (the forward one about 36 here); the
    smallest set, which the preconditioner does not fit, keeps BiCGSTAB."""
    import torch
    nd, S, u = _solver(gpu, kind, K, **kw)
    assert S.adjoint_info() == {"pressure_steps": 0, "viscous_iters": 0, "fallbacks": 0}
    st = S.new_state(u, torch.zeros_like(u))
    S.step(st, 2)
    adj = {k: to_dev(ri.random_vector(n, q) / n, gpu)
           for q, (k, n) in enumerate((("u", nd.n_v), ("v", nd.n_v), ("p_tilde", nd.n_p),
                                       ("cu_prev", nd.n_v), ("cv_prev", nd.n_v)))}
    grad = torch.zeros((2, nd.n_v), dtype=torch.float64, device=gpu)
    for _ in range(2):
        S.adjoint_step(st, adj, grad)
        info = S.adjoint_info()
        print(kind, K, kw, info, flush=True)
        assert info["fallbacks"] == 0 and info["viscous_iters"] > 0
        assert 0 < info["pressure_steps"] <= 100 if fast else info["pressure_steps"] == 0
    if not fast:
        import paper_2206_06495_amd as P
        with pytest.raises(P.RbfError):
            S.apply_precond_t(adj["p_tilde"])
    S.close()
