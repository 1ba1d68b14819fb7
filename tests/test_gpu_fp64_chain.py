"""Seeded FP64 Metropolis chains against the oracle's (positions, log|psi| and every
decision): networks just beyond the one-launch kernel, which move layer by layer with
the in-kernel generator, and the one-launch kernel with job boundaries inside a
workgroup and batches beyond its limit."""
import numpy as np
import pytest

from oracle import oracle as O
from paper_2401_10287_amd import inputs as I

pytestmark = pytest.mark.gpu


def _system(w1, w2, dets, spins, layers, nuclei):
    n = sum(spins)
    return I.System("S", np.array([[0.0, 0.3 * i, 1.9 * i] for i in range(nuclei)]), np.full(nuclei, 2.0), spins[0], spins[1],
                    layers, w1, w2, dets, 1, tuple(i % nuclei for i in range(n)), 1.0)


def _check(s, jobs, moves, group, pick=None):
    import torch
    from paper_2401_10287_amd import fnvmc
    cfg = fnvmc.Config(s, "fp64")
    th = I.init_params(s)
    B = sum(j[0] for j in jobs)
    x = I.init_walkers(s, B)
    tt, xt = torch.tensor(th, device="cuda"), torch.tensor(x, device="cuda")
    lp, _ = fnvmc.fn_log_psi(cfg, tt, xt)
    if group:
        acc = fnvmc.vmc_metropolis_step_group(cfg, tt, jobs, xt, lp, moves, 0.2)
    else:
        acc = fnvmc.vmc_metropolis_step(cfg, tt, xt, lp, moves, 0.2, seed=jobs[0][1], step0=jobs[0][2], stream_id=jobs[0][3])
    torch.cuda.synchronize()
    o, w0 = O.Oracle(s), 0
    for nb, seed, step0, sid in jobs:
        # (a walker's counters hold its index: the oracle takes the job's first walkers)
        m = nb if pick is None else min(nb, pick)
        xo, lo, ao = o.metropolis(th, x[w0:w0 + m], o.log_psi(th, x[w0:w0 + m])["log_abs"], moves, 0.2, seed=seed, step0=step0,
                                  stream_id=sid)
        np.testing.assert_array_equal(acc.cpu().numpy()[w0:w0 + m], ao)
        np.testing.assert_allclose(xt.cpu().numpy()[w0:w0 + m], xo, rtol=0, atol=1e-13)
        np.testing.assert_allclose(lp.cpu().numpy()[w0:w0 + m], lo, rtol=0, atol=1e-11)
        w0 += nb


JOBS = [(5, 3, 0, 1), (30, 5, 11, 2), (1, 3, 4, 9), (64, 2 ** 40 + 7, 2 ** 32 - 3, 4)]


# parameters beyond 64 KB, 5 electrons, and one determinant more than the one launch takes
@pytest.mark.parametrize("w1,w2,dets,spins,layers,nuclei", [(64, 8, 1, (1, 1), 1, 1), (16, 4, 2, (3, 2), 2, 2),
                                                            (16, 4, 17, (2, 1), 2, 1)])
@pytest.mark.parametrize("group", [False, True])
def test_layered_chain(w1, w2, dets, spins, layers, nuclei, group):
    _check(_system(w1, w2, dets, spins, layers, nuclei), JOBS if group else [(100, 2 ** 40 + 7, 2 ** 32 - 3, 4)], 8, group)


# one, two and four walkers of a workgroup; job boundaries inside workgroups
@pytest.mark.parametrize("extra", [0, 213, 700])
@pytest.mark.parametrize("w1,w2,dets,spins,nuclei", [(20, 6, 3, (2, 1), 2), (12, 5, 16, (0, 4), 1)])
def test_one_launch_chain(w1, w2, dets, spins, nuclei, extra):
    _check(_system(w1, w2, dets, spins, 2, nuclei), JOBS + ([(extra, 6, 1, 5)] if extra else []), 8, True)


# the batch limit of a plain call (four rounds: 12288 walkers of helium's network, 2048
# where one walker fits a workgroup) and one walker beyond it
@pytest.mark.parametrize("w1,w2,dets,spins,nuclei,limit", [(32, 8, 2, (1, 1), 1, 12288), (37, 4, 6, (2, 2), 2, 2048)])
@pytest.mark.parametrize("over", [0, 1])
def test_batch_limit(w1, w2, dets, spins, nuclei, limit, over):
    _check(_system(w1, w2, dets, spins, 2, nuclei), [(limit + over, 3, 1, 2)], 3, False, pick=50)
