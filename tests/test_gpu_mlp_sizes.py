"""GPU: the network's forward and backward kernels over batch sizes at the
edges of their tiles (16 samples, two tiles a workgroup), with inputs that
saturate the output clamp, against the FP64 network of the oracle.

Tolerance: 64 + 64 + 27 FP32 products in sequence bound the relative rounding
of a value by 155 x 2^-24 = 9.3e-6 of the sum of absolute terms; on the norms
compared here the terms cancel by less than a factor of two: 2e-5.
"""
import numpy as np
import pytest

from oracle import learned
from paper_1907_06696_amd import mfgmg
from tests.parity_cases import rel_err

pytestmark = pytest.mark.gpu

TOL = 2e-5


@pytest.mark.parametrize("n", [1, 3, 15, 16, 17, 31, 32, 33, 47, 64, 65, 1000, 4096, 40001])
def test_mlp_sizes(n):
    import torch
    torch.cuda.set_device(0)
    r = np.random.default_rng(n)
    w = r.uniform(-1, 1, 6147) * 0.35
    x = r.uniform(-1.5, 1.5, (n, 27))
    dy = r.uniform(-1, 1, (n, 3))
    w, x, dy = (a.astype(np.float32) for a in (w, x, dy))
    y_ref, cache_ref = learned.mlp_forward(w.astype(np.float64), x.astype(np.float64))
    dev = [torch.tensor(a, device="cuda") for a in (w, x, dy)]
    y, cache = mfgmg.mlp_forward(dev[0], dev[1])
    z1, z2, z3 = cache_ref[1], cache_ref[3], cache_ref[5]
    got = cache.double().cpu().numpy()
    assert rel_err(y.double().cpu().numpy(), y_ref) < TOL
    for a, b in ((got[:, :64], z1), (got[:, 64:128], z2), (got[:, 128:], z3)):
        assert rel_err(a, b) < TOL
    # the clamp's edge: a sample whose z3 rounds to the other side changes dw by
    # its whole share, so samples within rounding of it carry no gradient
    dy_ok = np.where(np.abs(np.abs(z3) - 2.0) < 1e-3, 0.0, dy).astype(np.float32)
    dw_ref = learned.mlp_backward(w.astype(np.float64), cache_ref, dy_ok.astype(np.float64))
    dw = mfgmg.mlp_backward(dev[0], dev[1], cache, torch.tensor(dy_ok, device="cuda"))
    assert rel_err(dw.double().cpu().numpy(), dw_ref) < TOL
