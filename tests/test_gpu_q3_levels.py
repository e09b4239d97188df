"""GPU: the Q3 operator's update forms on both sides of its size rule (the fused
kernel of levels up to 16^3, the brick and halo kernels of 32^3): accumulation
and the smoother from zero and from a start, inputs nonzero on the boundary,
outputs poisoned, against the oracle's Chebyshev recurrence on the library's
own FP64 operator (held to the oracle elsewhere).  Tolerances: the operator's
and smoother's 1e-12 (FP64) and 1e-5 (FP32) relative.
"""
import numpy as np
import pytest

from oracle import multigrid as omg
from paper_1907_06696_amd import inputs, mfgmg
from tests.parity_cases import rel_err

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def solver():
    import torch
    torch.cuda.set_device(0)
    s = mfgmg.Solver(5)
    s.set_element(2)
    s.finalize_mesh()
    qp = s.leaf_quadrature_points().reshape(-1, 3)
    s.set_viscosity(inputs.sinker_mu(qp, inputs.sinker_centres(8, 2), 1e4).reshape(-1, 64))
    yield s
    s.close()


@pytest.mark.parametrize("dtype,tol", [("float64", 1e-12), ("float32", 1e-5)])
@pytest.mark.parametrize("level", [4, 5])
def test_updates(solver, level, dtype, tol):
    import torch
    s, dt = solver, getattr(torch, dtype)
    n = s.info()["n_u"][level]
    m = 3 * (1 << level) + 1
    at = np.arange(m)
    inner = (at > 0) & (at < m - 1)
    free = np.repeat((inner[:, None, None] & inner[None, :, None] & inner[None, None, :]).ravel(), 3)
    x, y0, b = (inputs.uniform_vector(n, k).astype(dtype).astype(np.float64) for k in (11, 12, 13))

    def dev(v, d=dt):
        return torch.tensor(v, device="cuda", dtype=d)

    def A(v):
        y = torch.full((n,), float("nan"), device="cuda", dtype=torch.float64)
        s.vmult(level, dev(v, torch.float64), y)
        return y.cpu().numpy()

    ax = A(x)
    y = torch.full((n,), float("nan"), device="cuda", dtype=dt)
    s.vmult(level, dev(x), y)
    yh = y.double().cpu().numpy()
    assert rel_err(yh, ax) <= tol and np.array_equal(yh[~free], x[~free])
    y = dev(y0)
    s.vmult_add(level, dev(x), y)
    yh = y.double().cpu().numpy()
    assert rel_err(yh, y0 + np.where(free, ax, 0.0)) <= tol and np.array_equal(yh[~free], y0[~free])
    minv = torch.empty(n, device="cuda", dtype=torch.float64)
    s.inverse_diagonal(level, minv)
    minv = minv.cpu().numpy()
    for zero in (True, False):
        ref = omg.chebyshev(A, minv, b, None if zero else x, s.smoother_lambda(level), x_is_zero=zero)
        y = torch.full((n,), float("nan"), device="cuda", dtype=dt) if zero else dev(x)
        s.smooth(level, dev(b), y, x_is_zero=zero)
        assert rel_err(y.double().cpu().numpy(), ref) <= tol, zero
