"""Charges beyond 16 bits: raising every dot's continuous minimum by a whole number of
carriers raises its charge by as much and changes nothing else (ground states, softargmin
and adjoint, every scorer)."""
import numpy as np
import pytest
import torch

from paper_2404_04994_amd import workloads as W

pytestmark = pytest.mark.gpu
RAISE = 50000  # (times 16 dots: below the 10^6 carriers of a closed array)


@pytest.fixture(scope="module")
def qa():
    from paper_2404_04994_amd import qarray
    qarray.load()
    return qarray


def inputs(n_dot):
    d = W.grid4x4(310, npix=2)
    cdd = d.cdd[:n_dot, :n_dot].copy()
    # multiples of 2^-20, so that x_u is exact with and without the raise, and no dot is
    # held at zero
    x = np.random.default_rng(n_dot).integers(3 << 20, 6 << 20, (200, n_dot)) / 2.0 ** 20
    return cdd, np.eye(n_dot), torch.as_tensor(x).cuda(), torch.as_tensor(x + RAISE).cuda()


@pytest.mark.parametrize("closed,t", [(False, 1.0), (False, 0.5), (True, 1.0)])
@pytest.mark.parametrize("precision,exhaustive", [("fp64", False), ("fp64", True),
                                                  ("bf16x3", False), ("fp32", True)])
@pytest.mark.parametrize("n_dot", [4, 8, 9, 12, 16])
def test_ground_state(qa, n_dot, precision, exhaustive, closed, t):
    cdd, cgd, V, Vr = inputs(n_dot)
    kw = dict(closed=closed, t=t, precision=precision, exhaustive=exhaustive)
    n = qa.ground_state(cdd, cgd, V, nhat=4 * n_dot if closed else 0, **kw)
    nr = qa.ground_state(cdd, cgd, Vr, nhat=(4 + RAISE) * n_dot if closed else 0, **kw)
    assert torch.equal(nr, n + RAISE)


@pytest.mark.parametrize("closed", [False, True])
@pytest.mark.parametrize("kT", [0.05, 1e-4])  # (matrix form from 9 dots on, and the walk)
@pytest.mark.parametrize("n_dot", [4, 8, 9, 12, 16])
def test_softargmin_and_adjoint(qa, n_dot, kT, closed):
    """The closed arrays' constraint force brings in energies of some 10^5, whose rounding
    (2^-35) over kT bounds what may differ."""
    cdd, cgd, V, Vr = inputs(n_dot)
    kw, kr = dict(closed=closed, nhat=4 * n_dot if closed else 0), dict(
        closed=closed, nhat=(4 + RAISE) * n_dot if closed else 0)
    tol = 64 * 2.0 ** -35 / kT if closed else 1e-12 / kT
    nb, sv = qa.soft_charge(cdd, cgd, V, kT, **kw)
    nr, sr = qa.soft_charge(cdd, cgd, Vr, kT, **kr)
    assert (nr - RAISE - nb).abs().max() < max(tol, 1e-10)
    if n_dot > 12:
        return
    g = torch.as_tensor(np.random.default_rng(1).standard_normal(tuple(nb.shape))).cuda()
    dC, _, dV = qa.soft_charge_backward(cdd, cgd, V, kT, g, sv, **kw)
    rC, _, rV = qa.soft_charge_backward(cdd, cgd, Vr, kT, g, sr, **kr)
    scale = float(dV.abs().max()) + 1.0 / kT
    assert (rV - dV).abs().max() < max(tol, 1e-10) * scale * n_dot
