"""Softargmin of 9 dots and more at temperatures near the ends of the range, where the
averages are known: every admissible candidate weighs the same (hot), or the ground state
is all that counts (cold)."""
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


@pytest.mark.parametrize("kT", [1e250, 1e289, 1e295, 1e300, 1e305, 1.7e308])
@pytest.mark.parametrize("n_dot", [9, 12, 14])
def test_hot_thresholded(qa, n_dot, kT):
    """Open array, t = 1/2: a dot whose continuous minimum lies within 1/4 of a half-integer
    takes both roundings with equal weight, the others the nearest charge."""
    d = W.grid4x4(295, npix=2)
    cdd, cgd = d.cdd[:n_dot, :n_dot].copy(), d.cgd[:n_dot, :n_dot].copy()
    rng = np.random.default_rng(n_dot)
    x = rng.integers(1, 4, (50, n_dot)) + rng.uniform(0.05, 0.95, (50, n_dot))
    x[np.abs(np.abs(x % 1 - 0.5) - 0.25) < 1e-3] += 0.01
    V = np.linalg.solve(cgd, x.T).T.copy()
    nb, saved = qa.soft_charge(cdd, cgd, torch.as_tensor(V).cuda(), kT, t=0.5)
    f = np.floor(x)
    want = np.where(np.abs(x - f - 0.5) <= 0.25, f + 0.5, np.round(x))
    assert np.abs(nb.cpu().numpy() - want).max() < 1e-12


@pytest.mark.parametrize("kT", [1e-250, 1e-300, 1e-307, 1e-310, 5e-324])
@pytest.mark.parametrize("n_dot", [9, 12, 16])
def test_cold_uncoupled(qa, n_dot, kT):
    """Dots that nothing couples: every one takes its nearest charge."""
    rng = np.random.default_rng(n_dot)
    x = rng.integers(0, 4, (50, n_dot)) + rng.choice([0.2, 0.8], (50, n_dot))
    nb, _ = qa.soft_charge(np.eye(n_dot), np.eye(n_dot), torch.as_tensor(x).cuda(), kT)
    assert (nb.cpu().numpy() == np.round(x)).all()
