"""FP64 results do not depend on the batch: a job's moves in a group are bitwise
those of a group of its own and of vmc_metropolis_step with the split-reduction
products off, and a walker's local energy and log|psi| are bitwise those it gets
in a small batch, on both sides of the rules that choose kernels by rows."""
import pytest

from paper_2401_10287_amd import inputs as I

pytestmark = pytest.mark.gpu


def _group_equals_alone_and_plain(s, jobs, moves):
    import torch
    from paper_2401_10287_amd import fnvmc
    cfg = fnvmc.Config(s, "fp64")
    tt = torch.tensor(I.init_params(s), device="cuda")
    B = sum(j[0] for j in jobs)
    x0 = torch.tensor(I.init_walkers(s, B), device="cuda")
    lp0, _ = fnvmc.fn_log_psi(cfg, tt, x0)
    xg, lg = x0.clone(), lp0.clone()
    ag = fnvmc.vmc_metropolis_step_group(cfg, tt, jobs, xg, lg, moves, 0.2)
    w0 = 0
    for nb, seed, step0, sid in jobs:
        sl = slice(w0, w0 + nb)
        xa, la = x0[sl].clone(), lp0[sl].clone()
        aa = fnvmc.vmc_metropolis_step_group(cfg, tt, [(nb, seed, step0, sid)], xa, la, moves, 0.2)
        xp, lpp = x0[sl].clone(), lp0[sl].clone()
        try:
            fnvmc.fn_tuning_set("gemm_splitk", 0)
            ap = fnvmc.vmc_metropolis_step(cfg, tt, xp, lpp, moves, 0.2, seed=seed, step0=step0, stream_id=sid)
            torch.cuda.synchronize()
        finally:
            fnvmc.fn_tuning_set("gemm_splitk", 1)
        for got, alone, plain, what in ((xg[sl], xa, xp, "x"), (lg[sl], la, lpp, "log|psi|"), (ag[sl], aa, ap, "accepted")):
            assert torch.equal(got, alone), (nb, what)
            assert torch.equal(got, plain), (nb, what)
        w0 += nb
    assert 0 < ag.sum().item() < moves * B


# 256-wide layers: a 256-walker job has 32 tiles of 128 x 64 per product (the
# small-grid kernel's side), the group 288 (the tiled kernel's)
def test_group_of_lih():
    _group_equals_alone_and_plain(I.lih(), [(256, 3, 0, 1), (37, 5, 11, 2), (1024, 3, 4, 9), (963, 8, 2, 3)], 4)


# products of every layer on one side in the small batch, on the other in the large one
@pytest.mark.parametrize("w1,walkers", [(256, 700), (96, 3001)])
def test_energy_of_small_and_large_batches(w1, walkers):
    import dataclasses
    import torch
    from paper_2401_10287_amd import fnvmc
    s = dataclasses.replace(I.lih(), w1=w1)
    cfg = fnvmc.Config(s, "fp64")
    tt = torch.tensor(I.init_params(s), device="cuda")
    x = torch.tensor(I.init_walkers(s, walkers), device="cuda")
    big, lb, _ = fnvmc.fn_local_energy(cfg, tt, x)
    small, ls, _ = fnvmc.fn_local_energy(cfg, tt, x[-19:].contiguous())
    v, sg = fnvmc.fn_log_psi(cfg, tt, x)
    vs, ss = fnvmc.fn_log_psi(cfg, tt, x[-19:].contiguous())
    torch.cuda.synchronize()
    assert torch.isfinite(big).all()
    assert torch.equal(small, big[-19:]) and torch.equal(ls, lb[-19:])
    assert torch.equal(vs, v[-19:]) and torch.equal(ss, sg[-19:])


# networks that the one-launch kernel takes up to a batch limit, groups beyond it:
# 12288 walkers where four share a workgroup's parameters, 2048 where one fits
@pytest.mark.parametrize("w1,w2,dets,spins,nuclei,jobs", [
    (32, 8, 2, (1, 1), 1, [(256, 3, 0, 1), (37, 5, 11, 2), (12300, 3, 4, 9)]),
    (37, 4, 6, (2, 2), 2, [(100, 3, 0, 1), (256, 5, 11, 2), (2500, 3, 4, 9)])])
def test_group_of_a_small_network(w1, w2, dets, spins, nuclei, jobs):
    import numpy as np
    n = sum(spins)
    s = I.System("S", np.array([[0.0, 0.3 * i, 1.9 * i] for i in range(nuclei)]), np.full(nuclei, 2.0), spins[0], spins[1],
                 2, w1, w2, dets, 1, tuple(i % nuclei for i in range(n)), 1.0)
    _group_equals_alone_and_plain(s, jobs, 4)
