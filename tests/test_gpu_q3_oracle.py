"""GPU: the Q3 operator and its update forms on the largest level of the fused
kernel (16^3) and the smallest of the brick and halo kernels (32^3), against
the oracle's element matrix applied cell by cell: the operator, accumulation
and the smoother from zero and from a start, inputs nonzero on the boundary,
outputs poisoned.  Tolerances: the operator's and smoother's 1e-12 (FP64) and
1e-5 (FP32) relative, and the operator's row by row."""
import numpy as np
import pytest

from oracle import multigrid as omg, q3q2
from paper_1907_06696_amd import inputs, mfgmg
from tests.parity_cases import rel_err, row_err
from tests.test_gpu_parity import ROW32, ROW64
from tests.test_gpu_q3q2 import abs_bound

pytestmark = pytest.mark.gpu
LEAF = 5


class Level:
    """The oracle's level operator, matrix-free."""

    def __init__(self, level, mu):
        self.mesh, self.mu = q3q2.UniformMesh(level), mu
        self.dofs, self.free = self.mesh.cell_dofs(), self.mesh.free_dofs_mask()
        self.K, self.scale = q3q2.khat(), mu * self.mesh.h

    def apply(self, x):
        loc = (x * self.free)[self.dofs] @ self.K.T * self.scale[:, None]
        y = np.bincount(self.dofs.ravel(), weights=loc.ravel(), minlength=self.mesh.n_u)
        return np.where(self.free, y, x)

    def inverse_diagonal(self):
        d = np.bincount(self.dofs.ravel(), weights=(self.scale[:, None] * np.diag(self.K)).ravel(),
                        minlength=self.mesh.n_u)
        return np.where(self.free, 1.0 / d, 1.0)


@pytest.fixture(scope="module")
def setup():
    import torch
    torch.cuda.set_device(0)
    s = mfgmg.Solver(LEAF)
    s.set_element(2)
    s.finalize_mesh()
    qp = s.leaf_quadrature_points().reshape(-1, 3)
    mu_qp = inputs.sinker_mu(qp, inputs.sinker_centres(8, 2), 1e4).reshape(-1, 64)
    s.set_viscosity(mu_qp)
    n = 1 << LEAF
    mu = {LEAF: q3q2.harmonic_cell_viscosity(mu_qp)}   # coarser cells: the mean of their children
    mu[LEAF - 1] = mu[LEAF].reshape(n // 2, 2, n // 2, 2, n // 2, 2).mean(axis=(1, 3, 5)).ravel()
    yield s, {l: Level(l, m) for l, m in mu.items()}
    s.close()


@pytest.mark.parametrize("dtype,tol,row", [("float64", 1e-12, ROW64), ("float32", 1e-5, ROW32)])
@pytest.mark.parametrize("level", [LEAF - 1, LEAF])
def test_operator_and_updates(setup, level, dtype, tol, row):
    import torch
    s, levels = setup
    A, dt = levels[level], getattr(torch, dtype)
    n, free = A.mesh.n_u, A.free
    x, y0, b = (inputs.uniform_vector(n, k).astype(dtype).astype(np.float64) for k in (21, 22, 23))

    def dev(v):
        return torch.tensor(v, device="cuda", dtype=dt)

    def poisoned():
        return torch.full((n,), float("nan"), device="cuda", dtype=dt)

    def host(v):
        return v.double().cpu().numpy()

    ax = A.apply(x)
    y = poisoned()
    s.vmult(level, dev(x), y)
    e, r = rel_err(host(y), ax), row_err(host(y), ax, abs_bound(A.mesh, A.mu, x))
    print(f"[q3 oracle] level {level} {dtype}: rel {e:.2e} row {r:.2e}", flush=True)
    assert e <= tol and r <= row
    y = dev(y0)
    s.vmult_add(level, dev(x), y)
    assert rel_err(host(y), y0 + np.where(free, ax, 0.0)) <= tol and np.array_equal(host(y)[~free], y0[~free])
    for zero in (True, False):
        ref = omg.chebyshev(A.apply, A.inverse_diagonal(), b, None if zero else x, s.smoother_lambda(level),
                            x_is_zero=zero)
        y = poisoned() if zero else dev(x)
        s.smooth(level, dev(b), y, x_is_zero=zero)
        assert rel_err(host(y), ref) <= tol, zero
