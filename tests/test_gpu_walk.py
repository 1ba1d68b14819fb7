"""The walker-by-walker stream layer against the tiled one: the same products
in the same order, so a walker's local energy and log|psi| are bitwise those
it gets in a batch too small for that kernel (which the tiled kernel takes)."""
import dataclasses

import numpy as np
import pytest

from paper_2401_10287_amd import inputs as I

pytestmark = pytest.mark.gpu


def _system(spins, nuclei):
    n = sum(spins)
    s = I.h_chain(nuclei)
    return dataclasses.replace(s, n_up=spins[0], n_dn=spins[1], electron_site=tuple(i % nuclei for i in range(n)))


# rows per electron 3N + 2 at the edges of the 16-row blocks (17, 32, 35, 47,
# 50, 62), empty and uneven spins, features in one and in three steps of 32;
# batches with a partly empty last round
@pytest.mark.parametrize("spins,nuclei,prec,walkers", [((3, 2), 1, "bf16w", 250), ((5, 5), 8, "bf16w", 500),
                                                       ((8, 0), 2, "bf16w", 229), ((6, 5), 2, "bf16w", 147),
                                                       ((8, 7), 17, "bf16w", 300), ((8, 8), 2, "bf16x6", 150),
                                                       ((0, 11), 1, "bf16x6", 127), ((10, 10), 20, "bf16w", 413),
                                                       ((10, 10), 24, "bf16x6", 77)])
def test_walking_layer_bitwise(spins, nuclei, prec, walkers):
    import torch
    from paper_2401_10287_amd import fnvmc
    s = _system(spins, nuclei)
    cfg = fnvmc.Config(s, prec)
    tt = torch.tensor(I.init_params(s), dtype=torch.float32, device="cuda")
    x = torch.tensor(I.init_walkers(s, walkers), device="cuda")
    pick = torch.tensor(sorted({0, 1, 7, walkers // 2, walkers - 2, walkers - 1}), device="cuda")
    fnvmc.fn_tuning_set("gemm_splitk", 0)       # the other products' arithmetic then does not depend on the batch
    try:
        e, lp, _ = fnvmc.fn_local_energy(cfg, tt, x)
        e2, lp2, _ = fnvmc.fn_local_energy(cfg, tt, x[pick].contiguous())
        torch.cuda.synchronize()
    finally:
        fnvmc.fn_tuning_set("gemm_splitk", 1)
    assert bool(torch.isfinite(e).any())
    np.testing.assert_array_equal(e[pick].cpu().numpy(), e2.cpu().numpy())
    np.testing.assert_array_equal(lp[pick].cpu().numpy(), lp2.cpu().numpy())
