"""GPU: B u and B^T p on uniform leaves of 2^3 to 64^3 cells (below, at and
beyond the 33-column tile of the divergence), inputs nonzero on the boundary,
outputs poisoned beforehand, against the oracle's element matrix summed cell by
cell.  Tolerance: the block operators' 1e-12 relative.
"""
import numpy as np
import pytest

from oracle import operators as ops
from paper_1907_06696_amd import inputs
from tests.parity_cases import Case, rel_err

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("base", [1, 2, 3, 4, 5, 6])
def test_uniform_blocks(base):
    import torch
    torch.cuda.set_device(0)
    c = Case(base=base, sinkers=2, dr=10.0, seed=3)
    c.s.set_viscosity(c.mu_qp_lib)
    n_u, n_p = c.info["n_u"][c.L], c.info["n_p"]
    B = ops.CellwiseB(c.H.leaf)
    perm, pperm = c.dof_perm(c.L), c.pnode_perm()
    u, p = inputs.uniform_vector(n_u, 1), inputs.uniform_vector(n_p, 2)
    po = torch.full((n_p,), float("nan"), device="cuda", dtype=torch.float64)
    c.s.apply_div(torch.tensor(u[perm], device="cuda"), po)
    assert rel_err(po.cpu().numpy(), B.matvec(u)[pperm]) < 1e-12
    uo = torch.full((n_u,), float("nan"), device="cuda", dtype=torch.float64)
    c.s.apply_grad(torch.tensor(p[pperm], device="cuda"), uo)
    assert rel_err(uo.cpu().numpy(), B.rmatvec(p)[perm]) < 1e-12
    c.close()
