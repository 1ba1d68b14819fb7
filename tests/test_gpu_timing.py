"""Kernel classes of the timing diagnostics: a small FP64 network's one launch counts
in a class of its own, a larger one's kernels in theirs."""
import pytest

from paper_2401_10287_amd import inputs as I

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("name,small", [("He", True), ("LiH", False)])
def test_classes_of_an_fp64_walk(name, small):
    import torch
    from paper_2401_10287_amd import fnvmc
    s = {"He": I.he, "LiH": I.lih}[name]()
    cfg = fnvmc.Config(s, "fp64")
    tt = torch.tensor(I.init_params(s), device="cuda")
    x = torch.tensor(I.init_walkers(s, 32), device="cuda")
    try:
        fnvmc.fn_timing_enable(True)
        fnvmc.fn_timing_reset()
        lp, _ = fnvmc.fn_log_psi(cfg, tt, x)
        fnvmc.vmc_metropolis_step(cfg, tt, x, lp, 3, 0.2, seed=1)
        launches = {k: fnvmc.fn_timing_read(k)[1] for k in fnvmc.KERNEL_CLASSES}
    finally:
        fnvmc.fn_timing_enable(False)
        fnvmc.fn_timing_reset()
    if small:
        assert launches.pop("small_net") == 2 and not any(launches.values())
    else:
        assert launches["small_net"] == 0
        assert launches["stream_gemm"] == 4 * s.n_layers and launches["propose"] == 3 and launches["pack"] == 2
