"""Ragged batch of closed, thresholded diagrams.  In a wave of 64 pixels some thresholds
double (a few up to the whole box) while the other pixels keep their first candidate set:
every pixel against the FP64 oracle, and nothing written between the diagrams' outputs."""
import numpy as np
import pytest
import torch

from paper_2404_04994_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def qa():
    from paper_2404_04994_amd import qarray
    qarray.load()
    return qarray


GAP = 16
SENTINEL = -77


def packed_with_gaps(qa, diagrams):
    """A Batch whose diagrams' outputs lie GAP elements apart, all set to SENTINEL."""
    b = qa.Batch(diagrams)
    b.out_offsets = b.out_offsets + GAP * (1 + np.arange(len(diagrams)))
    total = int(b.out_offsets[-1]) + diagrams[-1].P * diagrams[-1].n_dot + GAP
    b.n = torch.full((total,), SENTINEL, dtype=torch.int32, device="cuda")
    b.nbar = torch.full((total,), float(SENTINEL), dtype=torch.float64, device="cuda")
    return b


@pytest.mark.parametrize("t", [0.4, 0.1])
@pytest.mark.parametrize("seeds", [(3, 5, 10, 16, 20, 26, 28), (0, 31, 35, 40, 41, 43, 54), (14,)])
def test_closed_thresholded_pixels(qa, oracle, seeds, t):
    ds = [W.ragged_diagram(31000 + s, npix=40) for s in seeds]
    assert all(d.closed for d in ds)
    for d in ds:
        d.t = t
    b = packed_with_gaps(qa, ds)
    st = b.run(stats=True)
    n_all, s_all = b.n.cpu().numpy(), b.nbar.cpu().numpy()
    free = np.ones(len(n_all), bool)
    for i, d in enumerate(ds):
        o = int(b.out_offsets[i])
        free[o:o + d.P * d.n_dot] = False
        n, nbar = b.result(i)
        ref = oracle.method_gs(d.cdd, d.cgd, d.V, closed=True, nhat=d.nhat, t=t)
        excl = (ref["e2"] - ref["e1"] < 1e-9) | ((ref["info"] & oracle.INFO_AMBIGUOUS) > 0)
        assert (n.sum(1) == d.nhat).all(), i
        assert ((n == ref["n"]).all(1) | excl).all(), i
        if d.kT > 0:
            rs, _, _ = oracle.method_soft(d.cdd, d.cgd, d.V, closed=True, nhat=d.nhat, t=t, kT=d.kT)
            assert np.abs(nbar - rs)[~excl].max() <= 1e-5, i
    assert (n_all[free] == SENTINEL).all() and (s_all[free] == SENTINEL).all()
    assert st["doubled_pixels"] > 0 or ds[0].n_dot < 4
