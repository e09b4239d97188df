"""GPU: the fused kernels of the small uniform levels (2^3 to 32^3 cells), with
u = 0 and, through node and cell maps, with u . n = 0 (free boundary nodes).

One mesh of 32^3 cells, every level of it: the operator, the accumulating
operator, and the smoother from zero and from a start, with inputs that are
nonzero on the boundary (identity rows), against the oracle.  Tolerances are
those of the other operator and smoother tests: 1e-12 (FP64) and 1e-5 (FP32)
relative; FP32 keeps 24 bits through at most four operator applications on a
smoother whose polynomial does not amplify.
"""
import numpy as np
import pytest

from oracle import multigrid as omg
from paper_1907_06696_amd import inputs
from tests.parity_cases import Case, rel_err

pytestmark = pytest.mark.gpu

TOL = {"float64": 1e-12, "float32": 1e-5}


@pytest.fixture(scope="module", params=["dirichlet", "noflux"])
def bc(request):
    return request.param


@pytest.fixture(scope="module")
def case(bc):
    import torch
    torch.cuda.set_device(0)
    c = Case(base=5, sinkers=6, dr=1e4, seed=4, bc=bc)
    c.s.set_viscosity(c.mu_qp_lib)
    yield c, omg.GMG(c.H, c.mus)
    c.close()


@pytest.mark.parametrize("dtype", ["float64", "float32"])
@pytest.mark.parametrize("level", [1, 2, 3, 4, 5])
def test_small_uniform_level(case, level, dtype):
    import torch
    c, g = case
    dt = getattr(torch, dtype)
    n = c.info["n_u"][level]
    perm = c.dof_perm(level)
    free = g.free[level]
    x, y0, b = (inputs.uniform_vector(n, s) for s in (11, 12, 13))

    def dev(v):
        return torch.tensor(v[perm], device="cuda", dtype=dt)

    def host(t):
        out = np.empty(n)
        out[perm] = t.double().cpu().numpy()
        return out

    ax = g.A[level] @ x
    y = torch.full((n,), float("nan"), device="cuda", dtype=dt)
    c.s.vmult(level, dev(x), y)
    assert rel_err(host(y), ax) < TOL[dtype]
    y = dev(y0)
    c.s.vmult_add(level, dev(x), y)
    assert rel_err(host(y), y0 + np.where(free, ax, 0.0)) < TOL[dtype]
    if level == 1:   # the coarse level has no smoother
        return
    for zero in (True, False):
        ref = omg.chebyshev(lambda v: g.A[level] @ v, g.minv[level], b, x, g.lam[level], x_is_zero=zero)
        y = torch.full((n,), float("nan"), device="cuda", dtype=dt) if zero else dev(x)
        c.s.smooth(level, dev(b), y, x_is_zero=zero)
        assert rel_err(host(y), ref) < TOL[dtype]
