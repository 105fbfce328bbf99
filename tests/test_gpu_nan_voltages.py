"""Voltages that are not numbers (9 dots and more): such a pixel's ground state is the
exhaustive scorer's (no charge), its softargmin is not a number, its gap is not counted,
and the other pixels do not notice."""
import numpy as np
import pytest
import torch

from paper_2404_04994_amd import build as B
from paper_2404_04994_amd import workloads as W


def test_files_that_promise_nans_honour_them():
    for name in ("qa_kernels.hip", "qa_rows.hip", "qa_soft.hip"):
        assert "-fno-honor-nans" not in B.FLAGS + B.PER_FILE.get(name, [])


def inputs(n_dot):
    d = W.grid4x4(280 + n_dot, npix=2)
    cdd, cgd = d.cdd[:n_dot, :n_dot].copy(), d.cgd[:n_dot, :n_dot].copy()
    V = np.random.default_rng(n_dot).uniform(-1.0, 3.0, (300, n_dot))
    W_ = V.copy()
    lost = np.array([0, 5, 16, 17, 63, 64, 130, 299])
    W_[lost, lost % n_dot] = np.nan
    keep = np.setdiff1d(np.arange(300), lost)
    return cdd, cgd, torch.as_tensor(V).cuda(), torch.as_tensor(W_).cuda(), lost, keep


@pytest.mark.gpu
@pytest.mark.parametrize("closed,t", [(False, 1.0), (False, 0.5), (True, 1.0), (True, 0.5)])
@pytest.mark.parametrize("n_dot", [9, 12, 14, 16])
def test_ground_state(n_dot, closed, t):
    from paper_2404_04994_amd import qarray as qa
    cdd, cgd, V, Vn, lost, keep = inputs(n_dot)
    kw = dict(closed=closed, nhat=n_dot if closed else 0, t=t)
    ref = qa.ground_state(cdd, cgd, V, **kw).cpu().numpy()
    n, st = qa.ground_state(cdd, cgd, Vn, stats=True, **kw)
    ne, se = qa.ground_state(cdd, cgd, Vn, stats=True, exhaustive=True, **kw)
    n = n.cpu().numpy()
    assert (n[keep] == ref[keep]).all()
    assert (n[lost] == 0).all() and (n == ne.cpu().numpy()).all()
    assert st["fp64_gap_below_1e9"] == se["fp64_gap_below_1e9"] == 0


@pytest.mark.gpu
@pytest.mark.parametrize("closed,t", [(False, 1.0), (False, 0.5), (True, 1.0), (True, 0.5)])
@pytest.mark.parametrize("n_dot", [9, 12, 14, 16])
def test_softargmin(n_dot, closed, t):
    from paper_2404_04994_amd import qarray as qa
    cdd, cgd, V, Vn, lost, keep = inputs(n_dot)
    kw = dict(closed=closed, nhat=n_dot if closed else 0, t=t)
    ref, _ = qa.soft_charge(cdd, cgd, V, 0.02, **kw)
    nb, _ = qa.soft_charge(cdd, cgd, Vn, 0.02, **kw)
    ref, nb = ref.cpu().numpy(), nb.cpu().numpy()
    assert (nb[keep] == ref[keep]).all()
    assert np.isnan(nb[lost]).all()
