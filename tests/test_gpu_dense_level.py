"""GPU: the 4^3 level's V-cycle as a dense matrix, and the dense coarse solve.

On a 4^3 leaf the whole V-cycle is that matrix; an adaptive mesh over it
uses it as its second level.  Both boundary conditions (81 and 225 coarse
dofs, 1,029 and 1,701 free dofs on the 4^3 level), both precisions, right-hand
sides that are nonzero on constrained dofs (whose rows are identities), and a
second viscosity on the same context.  Tolerances are the V-cycle tests' own:
1e-11 (FP64), 1e-4 (FP32).
"""
import numpy as np
import pytest

from oracle import multigrid as omg, operators as ops
from paper_1907_06696_amd import inputs
from tests.parity_cases import Case, rel_err

pytestmark = pytest.mark.gpu

TOL = {"float64": 1e-11, "float32": 1e-4}


@pytest.mark.parametrize("bc", ["dirichlet", "noflux"])
@pytest.mark.parametrize("corners", [(), ((1, 1, 1), (3, 0, 2))], ids=["uniform", "adaptive"])
def test_dense_level(bc, corners):
    import torch
    torch.cuda.set_device(0)
    c = Case(base=2, corners=corners, sinkers=3, dr=1e3, seed=7, bc=bc)
    L = c.L
    n = c.info["n_u"][L]
    perm = c.dof_perm(L)
    X = ops.gauss_points_of_cells(c.H.leaf).reshape(-1, 3)
    qp = c.s.leaf_quadrature_points().reshape(-1, 3)
    for centre_seed in (7, 8):   # the matrix follows the viscosity
        centres = inputs.sinker_centres(3, centre_seed)
        c.s.set_viscosity(inputs.sinker_mu(qp, centres, 1e3).reshape(-1, 27))
        mus = ops.level_viscosities(c.H, ops.harmonic_cell_viscosity(
            inputs.sinker_mu(X, centres, 1e3).reshape(-1, 27)))
        g = omg.GMG(c.H, mus)
        b = inputs.uniform_vector(n, 21)
        if corners:   # an adaptive leaf's transfers carry free dofs only
            b = b * g.free[L]
        ref = g.vcycle(b)
        perm1, b1 = c.dof_perm(1), inputs.uniform_vector(c.info["n_u"][1], 22)
        ref1 = g.coarse_solve(b1)
        for dtype, tol in TOL.items():
            dt = getattr(torch, dtype)
            x = torch.full((n,), float("nan"), device="cuda", dtype=dt)
            c.s.vcycle(torch.tensor(b[perm], device="cuda", dtype=dt), x)
            out = np.empty(n)
            out[perm] = x.double().cpu().numpy()
            assert rel_err(out, ref) < tol
            x = torch.full((len(b1),), float("nan"), device="cuda", dtype=dt)
            c.s.coarse_solve(torch.tensor(b1[perm1], device="cuda", dtype=dt), x)
            out = np.empty(len(b1))
            out[perm1] = x.double().cpu().numpy()
            assert rel_err(out, ref1) < tol
    c.close()
