"""FP64 jobs served in a gang have bitwise the results they have alone, with the
gang's total on the other side of the rules that choose kernels by rows."""
import numpy as np
import pytest

from paper_2401_10287_amd import inputs as I

pytestmark = pytest.mark.gpu


def _lih():
    return I.lih()


def _small():
    return I.System("S", np.array([[0.0, 0.0, 0.0], [0.0, 0.3, 1.9]]), np.full(2, 2.0), 2, 2, 2, 37, 4, 6, 1, (0, 1, 0, 1), 1.0)


@pytest.mark.parametrize("system,sizes", [(_lih, (128, 700, 256)), (_small, (256, 1900, 1700))])
def test_gang_equals_alone(system, sizes):
    import torch
    from paper_2401_10287_amd import fnvmc, serving
    s = system()
    cfg = fnvmc.Config(s, "fp64")
    th = torch.tensor(I.init_params(s), device="cuda")
    xs = [torch.tensor(I.init_walkers(s, b, seed=I.WALKER_SEED + 900 + k), device="cuda") for k, b in enumerate(sizes)]
    torch.cuda.synchronize()

    def serve(max_gang):
        srv = serving.Server(8 << 30, n_streams=1, quantum=4, max_gang=max_gang, gang_walkers=8192)
        ids = [srv.submit(cfg, th, x, 9, 0.2, seed=1, stream_id=k) for k, x in enumerate(xs)]
        srv.drain(ids)
        out = [srv.result(j) for j in ids]
        srv.close()
        return out

    alone, gang = serve(1), serve(8)
    assert [r["gang_jobs"] for r in alone] == [1] * 3 and [r["gang_jobs"] for r in gang] == [3] * 3
    for a, g in zip(alone, gang):
        assert a["state"] == g["state"] == "done"
        for key in ("mean", "variance", "std_error", "acceptance"):
            assert a[key] == g[key], key
