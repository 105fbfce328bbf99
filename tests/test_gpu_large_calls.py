"""Single calls whose setup takes 2^32 threads and more (a launch holds fewer): pixels
from all over the sweep, and its last ones, against a call on their voltages."""
import numpy as np
import pytest
import torch

from paper_2404_04994_amd import workloads as W

pytestmark = pytest.mark.gpu


# group of 2, 8 and 16 lanes per pixel: 2^32 threads are 1.88, 0.470 and 0.235 10^9 pixels
@pytest.mark.parametrize("n_dot,nx,ny", [(1, 46000, 41000), (5, 22000, 21400), (9, 16000, 14700)])
def test_more_threads_than_a_launch_holds(n_dot, nx, ny):
    from paper_2404_04994_amd import qarray as qa
    d = W.grid4x4(270, npix=2)
    cdd, cgd = d.cdd[:n_dot, :n_dot].copy(), d.cgd[:n_dot, :n_dot].copy()
    rng = np.random.default_rng(n_dot)
    sweep = dict(v0=rng.uniform(0.0, 2.0, n_dot), e1=rng.uniform(-0.5, 1.0, n_dot),
                 e2=rng.uniform(-0.5, 1.0, n_dot), a0=-1.0, a1=4.0, nx=nx, b0=-2.0, b1=3.0, ny=ny)
    qa.release()  # (the workspace of earlier tests)
    torch.cuda.empty_cache()
    n, st = qa.ground_state_grid(cdd, cgd, sweep, stats=True)
    assert st["pixels"] == nx * ny and st["qp_failures"] == 0
    p = np.concatenate([rng.integers(0, nx * ny, 4000), nx * ny - 1 - np.arange(1000)])
    a, b = np.linspace(-1.0, 4.0, nx)[p % nx], np.linspace(-2.0, 3.0, ny)[p // nx]
    V = sweep["v0"] + a[:, None] * sweep["e1"] + b[:, None] * sweep["e2"]
    few = qa.ground_state(cdd, cgd, torch.as_tensor(V).cuda())
    assert torch.equal(n[torch.as_tensor(p).cuda()], few)
    del n
    qa.release()
    torch.cuda.empty_cache()
