"""qa_time_kernels times the kernels that a call runs: one that scores as well up to 8 dots
(no time for a scorer), setup and scorer above."""
import pytest
import torch

from paper_2404_04994_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_dot", [2, 8, 12])
def test_kernels_of_a_call(n_dot):
    from paper_2404_04994_amd import qarray as qa
    d = W.double_dot(3, npix=30) if n_dot == 2 else W.grid4x4(3, npix=100)
    cdd, cgd = d.cdd[:n_dot, :n_dot].copy(), d.cgd[:n_dot].copy()
    V = torch.as_tensor(d.V).cuda()
    out = torch.full((d.P, n_dot), -1, dtype=torch.int32, device="cuda")
    setup, scorer = qa.time_kernels(cdd, cgd, V, out, 500)
    assert torch.equal(out, qa.ground_state(cdd, cgd, V))
    assert 0 < setup < 1.0
    if n_dot <= 8:
        assert scorer == 0.0
    else:
        assert 0 < scorer < 1.0
