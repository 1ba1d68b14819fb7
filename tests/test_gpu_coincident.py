"""Two electrons of one spin at one point (a node of psi, where the orbital
matrices have two equal columns): whether rounding leaves log|psi| finite must
not depend on the call, so the local energy's log|psi| is finite exactly where
fn_log_psi's is, for every spin size of the determinant kernels."""
import numpy as np
import pytest

from paper_2401_10287_amd import inputs as I

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("spins", [(2, 2), (3, 2), (4, 0), (5, 5), (6, 1), (7, 7), (8, 2), (9, 9), (10, 0), (10, 10), (11, 2)])
def test_coincident_electrons(spins, precision):
    import torch
    from paper_2401_10287_amd import fnvmc
    n, walkers = sum(spins), 200
    s = I.System("S", np.array([[0.0, 0.0, 0.0], [0.0, 0.0, 1.6]]), np.array([2.0, 1.0]), spins[0], spins[1], 2, 32, 8, 1,
                 walkers, tuple(i % 2 for i in range(n)), 1.0)
    cfg = fnvmc.Config(s, precision)
    x = I.init_walkers(s, walkers)
    x[::2, spins[0] - 1] = x[::2, 0]             # every other walker on a node
    tt = torch.tensor(I.init_params(s), dtype=cfg.param_dtype, device="cuda")
    xt = torch.tensor(x, device="cuda")
    _, le, _ = fnvmc.fn_local_energy(cfg, tt, xt)
    lv, _ = fnvmc.fn_log_psi(cfg, tt, xt)
    torch.cuda.synchronize()
    assert torch.isfinite(lv[1::2]).all()
    assert torch.equal(torch.isfinite(le), torch.isfinite(lv))
