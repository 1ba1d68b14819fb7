"""Determinants of the gradient's forward pass at every spin size of the
one-thread-per-matrix kernel and beyond it: entries of sum_p c_p d log|psi_p| / d
theta against the oracle with the FP64 tolerance of the gradient tests (1e-9 of
the largest entry)."""
import numpy as np
import pytest

from oracle import oracle as O
from paper_2401_10287_amd import inputs as I

pytestmark = pytest.mark.gpu


# each size 1 .. 11 once; 3 x 23 = 69 matrices leave the second workgroup partly empty
@pytest.mark.parametrize("spins", [(1, 2), (3, 4), (6, 5), (7, 8), (10, 9), (11, 0)])
def test_gradient_determinants(spins):
    import torch
    from paper_2401_10287_amd import fnvmc
    n, walkers = sum(spins), 23
    s = I.System("S", np.array([[0.0, 0.0, 0.0], [0.3, -0.4, 2.1]]), np.array([float(n), 1.0]), spins[0], spins[1], 2, 32, 8,
                 3, walkers, tuple(i % 2 for i in range(n)), 1.0)
    cfg = fnvmc.Config(s, "fp64")
    th, x = I.init_params(s), I.init_walkers(s, walkers)
    c = np.random.default_rng(3).standard_normal(walkers)
    g = fnvmc.fn_log_psi_vjp(cfg, torch.tensor(th, device="cuda"), torch.tensor(x, device="cuda"), torch.tensor(c, device="cuda"))
    torch.cuda.synchronize()
    idx = np.random.default_rng(4).choice(th.size, 30, replace=False)
    ref = c @ O.Oracle(s).dlogpsi_dtheta(th, x, idx)
    got = g.cpu().numpy()
    np.testing.assert_allclose(got[idx], ref, rtol=0, atol=1e-9 * np.abs(got).max())
