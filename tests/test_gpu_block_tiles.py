"""GPU: B u and B^T p on a uniform 128^3 leaf, where the divergence takes
several tiles along x (a wave's row holds up to 73 pressure points; 129 make two
tiles of 65, the last one partial) and its longest march (8 planes, the last one
a single plane).  Sampled rows against the oracle's element matrix summed over
the cells around a node: every x at a dozen (y, z), every z at three (x, y), and
random ones; inputs nonzero on the boundary, outputs poisoned beforehand.

Bound, row by row: 128 eps sum |B_ij| |u_j|, the sum cell by cell.  Along any
path from a u_j to its row the kernels round some 25 times (three one-axis
contractions with rounded weights, the scaling), the oracle some 120 times (a
27-point quadrature, a product of 81 terms, 8 cells), each half an eps."""
import numpy as np
import pytest

from oracle import fe
from paper_1907_06696_amd import inputs, mfgmg

pytestmark = pytest.mark.gpu
LEVEL = 7
EPS = np.finfo(np.float64).eps


def local_nodes(cells, order, m):
    """Lattice nodes [len(cells), (order + 1)^3] of the cells, x fastest."""
    a = np.arange((order + 1) ** 3)
    off = np.stack([a % (order + 1), a // (order + 1) % (order + 1), a // (order + 1) ** 2], 1)
    q = order * cells[:, None, :] + off[None]
    return q[..., 0] + m * (q[..., 1] + m * q[..., 2])


def check(got, rows):
    """rows: sums over cells of (selection, values, sums of absolute products)."""
    ref, bound = np.zeros(got.shape), np.zeros(got.shape)
    for sel, v, b in rows:
        ref[sel] += v
        bound[sel] += b
    err = np.abs(got - ref)
    print(f"  max error / bound {(err / np.maximum(128 * EPS * bound, 1e-300)).max():.3f}", flush=True)
    assert np.all(err <= 128 * EPS * bound)


def test_blocks_128_sampled_rows():
    import torch
    torch.cuda.set_device(0)
    n = 1 << LEVEL
    m, np1, h2 = 2 * n + 1, n + 1, 1.0 / n ** 2
    s = mfgmg.Solver(LEVEL)
    s.finalize_mesh()
    info = s.info()
    s.set_viscosity(np.ones((n ** 3, 27)))
    pkeys = s.support_points(LEVEL, 1)                        # X + m (Y + m Z) on the velocity lattice
    lat = (pkeys % m // 2) + np1 * (pkeys // m % m // 2 + np1 * (pkeys // (m * m) // 2))
    u, p = inputs.uniform_vector(info["n_u"][LEVEL], 1), inputs.uniform_vector(info["n_p"], 2)
    po = torch.full((info["n_p"],), float("nan"), device="cuda", dtype=torch.float64)
    s.apply_div(torch.tensor(u, device="cuda"), po)
    uo = torch.full((info["n_u"][LEVEL],), float("nan"), device="cuda", dtype=torch.float64)
    s.apply_grad(torch.tensor(p, device="cuda"), uo)
    po, uo = po.cpu().numpy(), uo.cpu().numpy().reshape(-1, 3)
    s.close()
    assert np.isfinite(po).all() and np.isfinite(uo).all()
    bhat = fe.element_matrices()[1]
    at = np.arange(m)
    wall = (at == 0) | (at == m - 1)
    fixed = (wall[:, None, None] | wall[None, :, None] | wall[None, None, :]).ravel()
    uf = np.where(fixed[:, None], 0.0, u.reshape(-1, 3))
    plat, out = np.empty(np1 ** 3), np.empty(np1 ** 3)
    plat[lat], out[lat] = p, po
    rng = np.random.default_rng(3)

    def points(side):
        line = np.arange(side)
        yz = np.concatenate([[[0, 0], [side - 1, side - 1], [1, side - 2]], rng.integers(0, side, (9, 2))])
        xy = np.concatenate([[[side // 2, side // 2 + 1]], rng.integers(0, side, (2, 2))])
        sets = [np.column_stack([line, np.full(side, a), np.full(side, b)]) for a, b in yz]
        sets += [np.column_stack([np.full(side, a), np.full(side, b), line]) for a, b in xy]
        return np.concatenate(sets + [rng.integers(0, side, (1500, 3))])

    corners = np.stack(np.meshgrid([0, 1], [0, 1], [0, 1], indexing="ij"), -1).reshape(-1, 3)
    P = points(np1)
    rows = []
    for d in corners:                                          # the cells P - d
        c = P - d
        sel = np.nonzero(((c >= 0) & (c < n)).all(1))[0]
        a = d[0] + 2 * d[1] + 4 * d[2]
        loc = uf[local_nodes(c[sel], 2, m)].reshape(len(sel), 81)
        rows.append((sel, h2 * (loc @ bhat[a]), h2 * (np.abs(loc) @ np.abs(bhat[a]))))
    check(out[P[:, 0] + np1 * (P[:, 1] + np1 * P[:, 2])], rows)
    X = points(m)
    node = X[:, 0] + m * (X[:, 1] + m * X[:, 2])
    rows = []
    for d in corners:                                          # the cell of the node, and the one below it on an edge
        c = X // 2 - d
        ok = ((c >= 0) & (c < n)).all(1) & ((d == 0) | (X % 2 == 0)).all(1) & ~fixed[node]
        sel = np.nonzero(ok)[0]
        l = X[sel] - 2 * c[sel]
        col = 3 * (l[:, 0] + 3 * (l[:, 1] + 3 * l[:, 2]))
        loc = plat[local_nodes(c[sel], 1, np1)]
        B = np.stack([bhat[:, col + q] for q in range(3)], -1)  # [8, rows, component]
        rows.append((sel, h2 * np.einsum("ra,arc->rc", loc, B), h2 * np.einsum("ra,arc->rc", np.abs(loc), np.abs(B))))
    check(uo[node], rows)
