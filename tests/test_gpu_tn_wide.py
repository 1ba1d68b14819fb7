"""Weight-gradient products of layers wider than 256, whose many tiles leave fewer
than eight row splits (1, 2 and 4 here): the FP64 gradient against the oracle with
the FP64 tolerance of the gradient tests (1e-9 of the largest entry), and the FP32
pretraining gradient (no determinants, so no amplification near nodes) against the
FP64 one, each tensor within 2^-15 of its norm: chains of up to 512 sums of rounding
2^-24 each."""
import numpy as np
import pytest

from oracle import oracle as O
from paper_2401_10287_amd import inputs as I

pytestmark = pytest.mark.gpu


def _system(w1, walkers):
    return I.System("S", np.array([[0.0, 0.0, 0.0], [0.5, 0.0, 1.9]]), np.array([2.0, 1.0]), 1, 1, 2, w1, 8, 2, walkers, (0, 1), 1.0)


# rows of a product: 2 x walkers (layers), walkers (spin means, head)
@pytest.mark.parametrize("w1,walkers", [(512, 300), (1024, 70)])
def test_fp64_gradient(w1, walkers):
    import torch
    from paper_2401_10287_amd import fnvmc
    s = _system(w1, walkers)
    th, x = I.init_params(s), I.init_walkers(s, walkers)
    rng = np.random.default_rng(walkers)
    c = rng.standard_normal(walkers)
    g = fnvmc.fn_log_psi_vjp(fnvmc.Config(s, "fp64"), torch.tensor(th, device="cuda"), torch.tensor(x, device="cuda"),
                             torch.tensor(c, device="cuda"))
    torch.cuda.synchronize()
    off = I.param_offsets(s)
    idx = np.concatenate([off[k][0] + rng.choice(int(np.prod(off[k][1])), 3, replace=False) for k in ("V0", "V1", "w_up", "w_dn")])
    ref = c @ O.Oracle(s).dlogpsi_dtheta(th, x, idx)
    got = g.cpu().numpy()
    np.testing.assert_allclose(got[idx], ref, rtol=0, atol=1e-9 * np.abs(got).max())


@pytest.mark.parametrize("w1,walkers", [(512, 300), (1024, 70), (1024, 1500)])
def test_fp32_pretraining_gradient(w1, walkers):
    import torch
    from paper_2401_10287_amd import fnvmc
    s = _system(w1, walkers)
    th = I.init_params(s).astype(np.float32)
    x = torch.tensor(I.init_walkers(s, walkers), device="cuda")
    tg = [torch.tensor(np.random.default_rng(q).standard_normal((walkers, 2, 1, 1)), device="cuda") for q in (0, 1)]
    _, g = fnvmc.fn_pretrain_grad(fnvmc.Config(s, "fp32"), torch.tensor(th, device="cuda"), x, *tg)
    _, r = fnvmc.fn_pretrain_grad(fnvmc.Config(s, "fp64"), torch.tensor(th.astype(np.float64), device="cuda"), x, *tg)
    torch.cuda.synchronize()
    g, r = g.double().cpu().numpy(), r.cpu().numpy()
    for name, (o, shape) in I.param_offsets(s).items():
        if name in ("V0", "V1", "w_up", "w_dn"):
            sl = slice(o, o + int(np.prod(shape)))
            assert np.linalg.norm(g[sl] - r[sl]) <= 2.0 ** -15 * np.linalg.norm(r[sl]), name
