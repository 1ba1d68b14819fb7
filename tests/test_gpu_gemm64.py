"""FP64 matrix-core products: local energy and gradient of log|psi| at sizes on
both sides of the small-grid rule and at widths that leave tiles partly empty,
against the oracle (FP64 tolerances of the parity and gradient tests)."""
import numpy as np
import pytest

from oracle import oracle as O
from paper_2401_10287_amd import inputs as I

pytestmark = pytest.mark.gpu


def _system(w1, w2, dets, spins, walkers):
    n = sum(spins)
    return I.System("S", np.array([[0.0, 0.0, 0.0], [0.0, 0.0, 1.9]]), np.array([2.0, 1.0]), spins[0], spins[1], 3, w1,
                    w2, dets, walkers, tuple(i % 2 for i in range(n)), 1.0)


# widths 20 (padded columns), 64 / 65 / 96 (one and two column tiles), 130 (a third
# 64-wide tile); walkers that give one row tile, and more than 256 tiles
@pytest.mark.parametrize("w1,w2,dets,spins,walkers", [(20, 6, 3, (2, 1), 1), (64, 8, 2, (1, 1), 37),
                                                      (65, 5, 2, (2, 2), 700), (96, 16, 5, (2, 1), 1300),
                                                      (130, 8, 16, (2, 2), 611)])
def test_fp64_products(w1, w2, dets, spins, walkers):
    import torch
    from paper_2401_10287_amd import fnvmc
    s = _system(w1, w2, dets, spins, walkers)
    th = I.init_params(s)
    x = I.init_walkers(s, walkers)
    cfg = fnvmc.Config(s, "fp64")
    tt = torch.tensor(th, device="cuda")
    e, lp, _ = fnvmc.fn_local_energy(cfg, tt, torch.tensor(x, device="cuda"))
    torch.cuda.synchronize()
    pick = np.unique(np.r_[0, walkers // 3, walkers // 2, walkers - 1])
    ref = O.Oracle(s).local_energy(th, x[pick])
    np.testing.assert_allclose(e.cpu().numpy()[pick], ref["e_loc"], rtol=0, atol=1e-7)
    np.testing.assert_allclose(lp.cpu().numpy()[pick], ref["log_abs"], rtol=1e-10)
    if w1 % 32 == 0:
        c = np.random.default_rng(1).standard_normal(4)
        g = fnvmc.fn_log_psi_vjp(cfg, tt, torch.tensor(x[:4], device="cuda"), torch.tensor(c, device="cuda"))
        torch.cuda.synchronize()
        idx = np.random.default_rng(2).choice(th.size, 40, replace=False)
        ref = c @ O.Oracle(s).dlogpsi_dtheta(th, x[:4], idx)
        got = g.cpu().numpy()
        np.testing.assert_allclose(got[idx], ref, rtol=0, atol=1e-9 * np.abs(got).max())
