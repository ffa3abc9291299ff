"""The lattice preconditioner at the sizes where its transform changes kernels (n = K - 1
lattice points a side: one launch for product and mode solves up to 64 and up to
128, two beyond; odd and even n, and the largest) against its plain statement, in FP64 and FP32."""
import pytest

import rbf_inputs as ri
from tests.helpers import rel_err, to_dev
from tests.test_gpu_parity import _gpu_solver, _lattice_precond_reference

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("n", [7, 8, 63, 64, 65, 126, 127, 128, 129, 256, 257, 512])
def test_transform_sizes(gpu, n, precision):
    import paper_2206_06495_amd as P
    K = n + 1
    nd = ri.cavity_nodes(K, 0.3, 4)
    S, ops, u_bc, v_bc = _gpu_solver(P, nd, gpu, 100.0, 1e-3, precond="lattice",
                                     precision=precision)
    y = ri.random_vector(nd.n_p, 11)
    z = S.apply_precond(to_dev(y, gpu)).cpu().numpy()
    S.close()
    # both grow with the condition number of the lattice solve, about 0.4 K^2
    tol = max(1e-12, 4e-16 * K * K) if precision == "fp64" else 2e-5 * max(1.0, (K / 40) ** 2)
    assert rel_err(z, _lattice_precond_reference(nd, ops, y)) <= tol
