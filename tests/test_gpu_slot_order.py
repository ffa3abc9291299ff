"""The solver's own copies of the operators are in column order: a solver given
stencils with permuted slots takes the same steps, bit for bit, for the compiled
stencil width and the generic one."""
import numpy as np
import pytest

import rbf_inputs as ri
from tests.helpers import to_dev, gpu_cavity_ops

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [28, 24, 32])
def test_permuted_slots_give_the_same_steps(gpu, n):
    import torch
    import paper_2206_06495_amd as P
    nd = ri.hex_cavity_nodes(14, 0.3, 1)
    grid, ops = gpu_cavity_ops(nd, gpu, n=n)
    gen = torch.Generator().manual_seed(3)
    mixed = {"k": n}
    for name in ("vv", "pv", "pp", "vp"):
        idx = ops["idx_" + name]
        perm = torch.argsort(torch.rand(idx.shape, generator=gen), dim=0).to(gpu)  # per row
        mixed["idx_" + name] = idx.gather(0, perm).contiguous()
        for what in ("dx", "dy", "lap"):
            if f"{name}_{what}" in ops:
                mixed[f"{name}_{what}"] = ops[f"{name}_{what}"].gather(0, perm).contiguous()
    u_bc, v_bc = ri.cavity_bc(nd.v_tag)
    out = []
    for o in (ops, mixed):
        S = P.Solver(grid, o, to_dev(u_bc, gpu), to_dev(v_bc, gpu), 100.0, 2e-3)
        st = S.new_state(to_dev(u_bc, gpu), to_dev(v_bc, gpu))
        S.step(st, 3)
        out.append(st)
        S.close()
    for key in ("u", "v", "p", "p_tilde", "cu_prev", "cv_prev"):
        assert torch.equal(out[0][key], out[1][key]), key
