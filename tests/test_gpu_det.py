"""The determinant stage over the spin sizes and counts at which its kernels
change, FP64, against the oracle: local energy within 1e-7 Ha per walker (the
FP64 tolerance of the parity tests) and log|psi| within 1e-10 relative."""
import numpy as np
import pytest

from oracle import oracle as O
from paper_2401_10287_amd import inputs as I

pytestmark = pytest.mark.gpu


# electrons per spin: each side of a kernel's range (2 / 3, 10 / 11, 12 / 13),
# odd and even, unequal; determinants 1, 3, 5; walkers that leave a workgroup of
# four partly empty; more than 64 directions with a second block of them
@pytest.mark.parametrize("spins,dets,walkers", [((3, 2), 3, 5), ((4, 4), 1, 9),
                                                     ((7, 3), 5, 3), ((0, 8), 3, 6),
                                                     ((5, 5), 16, 35), ((9, 10), 2, 4),
                                                     ((11, 7), 2, 3), ((12, 13), 2, 3),
                                                     ((10, 12), 2, 5)])
@pytest.mark.parametrize("iso", [False, True])
def test_determinant_sizes(spins, dets, walkers, iso):
    import torch
    from paper_2401_10287_amd import fnvmc
    n = sum(spins)
    xyz = np.array([[0.0, 0.0, 0.0], [0.3, -0.4, 2.1]])
    s = I.System("S", xyz, np.array([float(n), 1.0]), spins[0], spins[1], 2, 32, 8, dets, walkers,
                 tuple(i % 2 for i in range(n)), 1.0, int(iso))
    th = I.init_params(s)
    rng = np.random.default_rng(5)
    for name, v in I.view_params(s, th).items():
        if name.startswith(("pi_", "sig_")):
            v += 0.2 * rng.standard_normal(v.shape)
    x = I.init_walkers(s, walkers)
    cfg = fnvmc.Config(s, "fp64")
    tt = torch.tensor(th, dtype=cfg.param_dtype, device="cuda")
    xt = torch.tensor(x, device="cuda")
    e, lp, _ = fnvmc.fn_local_energy(cfg, tt, xt)
    v, sg = fnvmc.fn_log_psi(cfg, tt, xt)
    torch.cuda.synchronize()
    o = O.Oracle(s)
    ref = o.local_energy(tt.double().cpu().numpy(), x)
    np.testing.assert_allclose(e.cpu().numpy(), ref["e_loc"], rtol=0, atol=1e-7)
    np.testing.assert_allclose(lp.cpu().numpy(), ref["log_abs"], rtol=1e-10)
    np.testing.assert_allclose(v.cpu().numpy(), ref["log_abs"], rtol=1e-10)
