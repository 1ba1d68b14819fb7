"""Small-grid products and value-row layers: a walker's results do not depend on
the size of its batch while no reduction is split over waves, so a batch that
takes these kernels has to give the bits that the tiled kernels give in a batch
of another size."""
import numpy as np
import pytest

from paper_2401_10287_amd import inputs as I

pytestmark = pytest.mark.gpu


def _system(w1, spins):
    n = sum(spins)
    return I.System("S", np.array([[0.0, 0.0, 0.0], [0.0, 0.0, 1.9]]), np.array([4.0, 3.0]), spins[0], spins[1], 3, w1,
                    8, 2, 1, tuple(i % 2 for i in range(n)), 1.0)


# output widths just past one column block, past 64, and 256; rows that end inside
# a tile; one and several weight parts.  Rows per walker: 17.
@pytest.mark.parametrize("w1,precision,walkers", [(36, "bf16x6", 1001), (72, "bf16x6", 701), (100, "bf16w", 501),
                                                  (256, "bf16x3", 299), (256, "bf16w", 301), (256, "bf16w2", 300),
                                                  (72, "bf16", 703)])
def test_small_grid_products(w1, precision, walkers):
    import torch
    from paper_2401_10287_amd import fnvmc
    s = _system(w1, (3, 2))
    cfg = fnvmc.Config(s, precision)
    tt = torch.tensor(I.init_params(s), dtype=cfg.param_dtype, device="cuda")
    x = torch.tensor(I.init_walkers(s, 4000), device="cuda")
    try:
        fnvmc.fn_tuning_set("gemm_splitk", 0)        # the heads of the small batch too
        big, lb, _ = fnvmc.fn_local_energy(cfg, tt, x)
        small, ls, _ = fnvmc.fn_local_energy(cfg, tt, x[:walkers].contiguous())
        torch.cuda.synchronize()
    finally:
        fnvmc.fn_tuning_set("gemm_splitk", 1)
    assert torch.isfinite(small).all()
    assert torch.equal(small, big[:walkers]) and torch.equal(ls, lb[:walkers])
