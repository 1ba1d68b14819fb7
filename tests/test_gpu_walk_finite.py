"""The walking stream layer with six products and four row blocks, on both sides of
its batch rule: bitwise a small batch's results (the tiled kernel), every entry finite."""
import dataclasses

import pytest

from paper_2401_10287_amd import inputs as I

pytestmark = pytest.mark.gpu


# one round, 59% and 73% full, and two, 56% and 60%; features in one and in three steps
@pytest.mark.parametrize("spins,nuclei,prec,walkers", [((8, 8), 2, "bf16x6", 76), ((8, 8), 2, "bf16x6", 93),
                                                     ((10, 10), 24, "bf16x6", 93), ((9, 8), 1, "bf16x6", 144),
                                                     ((9, 8), 1, "bf16x6", 154), ((8, 7), 17, "bf16w", 300)])
def test_walking_layer_finite(spins, nuclei, prec, walkers):
    import torch
    from paper_2401_10287_amd import fnvmc
    s = dataclasses.replace(I.h_chain(nuclei), n_up=spins[0], n_dn=spins[1],
                            electron_site=tuple(i % nuclei for i in range(sum(spins))))
    cfg = fnvmc.Config(s, prec)
    tt = torch.tensor(I.init_params(s), dtype=torch.float32, device="cuda")
    x = torch.tensor(I.init_walkers(s, walkers), device="cuda")
    pick = torch.tensor([0, 7, walkers // 2, walkers - 1], device="cuda")
    fnvmc.fn_tuning_set("gemm_splitk", 0)       # the other products' arithmetic then does not depend on the batch
    try:
        e, lp, _ = fnvmc.fn_local_energy(cfg, tt, x)
        e2, lp2, _ = fnvmc.fn_local_energy(cfg, tt, x[pick].contiguous())
        torch.cuda.synchronize()
    finally:
        fnvmc.fn_tuning_set("gemm_splitk", 1)
    assert torch.isfinite(e).all() and torch.isfinite(lp).all()
    assert torch.equal(e[pick], e2) and torch.equal(lp[pick], lp2)
