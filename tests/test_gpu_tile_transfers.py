"""GPU: transfers of the levels that run tile by tile (coarse levels of 2^3 to
16^3 cells; u = 0, and u . n = 0 through the node maps), inputs nonzero on the
boundary, outputs poisoned, against the oracle's matrices.  Tolerances: a row
sums at most 125 products, so 125 u of the sum of magnitudes (FP64 1.4e-14, FP32
7.5e-6 relative to a vector norm).
"""
import numpy as np
import pytest

from oracle import multigrid as omg
from paper_1907_06696_amd import inputs
from tests.parity_cases import Case, rel_err

pytestmark = pytest.mark.gpu

TOL = {"float64": 1.4e-14, "float32": 7.5e-6}


@pytest.fixture(scope="module", params=["dirichlet", "noflux"])
def case(request):
    import torch
    torch.cuda.set_device(0)
    c = Case(base=5, sinkers=2, dr=10.0, seed=4, bc=request.param)
    c.s.set_viscosity(c.mu_qp_lib)
    yield c, omg.GMG(c.H, c.mus)
    c.close()


@pytest.mark.parametrize("dtype", ["float64", "float32"])
@pytest.mark.parametrize("level", [2, 3, 4, 5])
def test_tile_transfers(case, level, dtype):
    import torch
    c, g = case
    dt = getattr(torch, dtype)
    nf, nc = c.info["n_u"][level], c.info["n_u"][level - 1]
    pf, pc = c.dof_perm(level), c.dof_perm(level - 1)
    P = g.P[level]
    x = inputs.uniform_vector(nc, 51).astype(dtype).astype(np.float64)
    y = torch.full((nf,), float("nan"), device="cuda", dtype=dt)
    c.s.prolongate(level, torch.tensor(x[pc], device="cuda", dtype=dt), y)
    assert rel_err(y.double().cpu().numpy(), (P @ x)[pf]) <= TOL[dtype]
    r = inputs.uniform_vector(nf, 52).astype(dtype).astype(np.float64)
    y = torch.full((nc,), float("nan"), device="cuda", dtype=dt)
    c.s.restrict(level, torch.tensor(r[pf], device="cuda", dtype=dt), y)
    assert rel_err(y.double().cpu().numpy(), (P.T @ r)[pc]) <= TOL[dtype]
