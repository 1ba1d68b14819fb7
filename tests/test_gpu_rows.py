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


# value rows of the 256-wide layers: the first, middle and last layer's reductions
# (features of 2 and of 20 nuclei, pair means), rows that end inside a tile, fewer
# and more tiles than workgroups; the small batch is under the kernel's 4096 rows
@pytest.mark.parametrize("nuclei,spins,precision,walkers", [(2, (3, 2), "bf16w", 901), (2, (3, 2), "bf16x6", 820),
                                                            (20, (4, 3), "bf16w", 3001), (20, (4, 3), "bf16x6", 3003)])
def test_value_rows(nuclei, spins, precision, walkers):
    import torch
    from paper_2401_10287_amd import fnvmc
    n = sum(spins)
    s = I.System("S", np.array([[0.0, 0.1 * i, 1.4 * i] for i in range(nuclei)]), np.full(nuclei, 2.0), spins[0], spins[1],
                 3, 256, 32, 2, 1, tuple(i % nuclei for i in range(n)), 1.0)
    cfg = fnvmc.Config(s, precision)
    tt = torch.tensor(I.init_params(s), dtype=cfg.param_dtype, device="cuda")
    x = torch.tensor(I.init_walkers(s, walkers), device="cuda")
    try:
        fnvmc.fn_tuning_set("gemm_splitk", 0)
        big, sb = fnvmc.fn_log_psi(cfg, tt, x)
        tail, st = fnvmc.fn_log_psi(cfg, tt, x[-257:].contiguous())
        torch.cuda.synchronize()
    finally:
        fnvmc.fn_tuning_set("gemm_splitk", 1)
    assert torch.isfinite(big).all()
    assert torch.equal(tail, big[-257:]) and torch.equal(st, sb[-257:])
