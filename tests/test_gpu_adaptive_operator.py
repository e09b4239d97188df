"""GPU: the operator on adaptive levels whose leaf mixes 4^3 and 2^3 blocks,
single cells with and without hanging nodes (scattered refined cells leave
partial sibling groups: a few and more than one wave's 64 of each), into
poisoned outputs, on every level, against the oracle's matrix.  Tolerances: the
operator's 1e-12 (FP64) and 1e-5 (FP32) relative; identity rows exact.
"""
import numpy as np
import pytest

from oracle import multigrid as omg
from paper_1907_06696_amd import inputs
from tests.parity_cases import Case, rel_err

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("bc", ["dirichlet", "noflux"])
@pytest.mark.parametrize("base,scattered,times", [(2, 3, 2), (3, 9, 1), (4, 60, 1)])
def test_mixed_leaf(base, scattered, times, bc):
    import torch
    torch.cuda.set_device(0)
    n = 1 << base
    pick = np.random.default_rng(base).choice(n ** 3, size=scattered, replace=False)
    corners = [(int(i % n), int(i // n % n), int(i // n ** 2)) for i in pick]
    c = Case(base=base, corners=corners, times=times, dr=1e3, seed=4, bc=bc)
    c.s.set_viscosity(c.mu_qp_lib)
    gmg = omg.GMG(c.H, c.mus)
    for ell in range(1, c.L + 1):
        n_u = c.info["n_u"][ell]
        perm = c.dof_perm(ell)
        free = gmg.free[ell][perm]
        for dt, npt, tol in ((torch.float64, np.float64, 1e-12), (torch.float32, np.float32, 1e-5)):
            x = inputs.uniform_vector(n_u, 70 + ell).astype(npt).astype(np.float64)
            ref = (gmg.A[ell] @ x)[perm]
            y = torch.full((n_u,), float("nan"), device="cuda", dtype=dt)
            xd = torch.tensor(x[perm], device="cuda", dtype=dt)
            c.s.vmult(ell, xd, y)
            yh = y.double().cpu().numpy()
            assert rel_err(yh, ref) <= tol, (ell, dt)
            assert np.array_equal(yh[~free], x[perm][~free])
            c.s.vmult_add(ell, xd, y)
            assert rel_err(y.double().cpu().numpy()[free], 2.0 * ref[free]) <= tol, (ell, dt)
    c.close()
