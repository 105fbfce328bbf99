"""FP64 search in bound order (9 <= N <= 16) against the exhaustive FP64 scorer
of the same candidate sets.

Both score in FP64, so they return the same states; only where a runner-up lies
within 1e-9 (counted by both) may rounding choose, and there the two states'
energies have to agree.  Dot counts cover every number of high dots (3..10,
below and above one table of 64 high states), pixel counts one pixel, a partly
filled block, and more pixels than the chip holds waves."""
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


def sub_array(n, seed):
    d = W.grid4x4(seed, npix=2)
    return d.cdd[:n, :n].copy(), d.cgd[:n, :n].copy()


def check(qa, cdd, cgd, V, **kw):
    print("rows", cdd.shape[0], V.shape[0], kw, flush=True)
    Vd = torch.as_tensor(V).cuda()
    n, s = qa.ground_state(cdd, cgd, Vd, stats=True, **kw)
    ne, se = qa.ground_state(cdd, cgd, Vd, stats=True, exhaustive=True, **kw)
    n, ne = n.cpu().numpy(), ne.cpu().numpy()
    assert s["candidates"] == se["candidates"] == se["scored"]
    assert 0 < s["scored"]
    assert s["fp64_gap_below_1e9"] == se["fp64_gap_below_1e9"]
    diff = np.where((n != ne).any(1))[0]
    assert len(diff) <= s["fp64_gap_below_1e9"]
    if len(diff):
        A, xu = np.linalg.inv(cdd), V[diff] @ cgd.T
        e, f = n[diff] - xu, ne[diff] - xu
        assert np.abs(((e @ A) * e - (f @ A) * f).sum(1)).max() < 4e-9
    return n, s


@pytest.mark.parametrize("closed,t", [(False, 1.0), (False, 0.5), (True, 1.0), (True, 0.4)])
@pytest.mark.parametrize("n_dot", range(9, 17))
def test_rows_equal_exhaustive(qa, n_dot, closed, t):
    pixels = {9: 1, 10: 7, 11: 65, 12: 4099, 13: 513, 14: 130, 15: 300, 16: 700}[n_dot]
    rng = np.random.default_rng(1000 + n_dot)
    kw = dict(closed=closed, nhat=n_dot if closed else 0, t=t)
    for cdd, cgd in (sub_array(n_dot, 260), W.random_maxwell(n_dot, 900 + n_dot)):
        # from far below zero (the QP) to several charges per dot
        check(qa, cdd, cgd, rng.uniform(-3.0, 4.0, (pixels, n_dot)), **kw)


def test_rows_many_pixels(qa):
    cdd, cgd = sub_array(9, 261)
    V = np.random.default_rng(7).uniform(-1.0, 3.0, (70001, 9))
    check(qa, cdd, cgd, V)


@pytest.mark.parametrize("closed", [False, True])
def test_rows_exact_ties(qa, closed):
    """Identical dots on a symmetric sweep: many degenerate minima."""
    n = 12
    cdd = np.full((n, n), -0.05) + np.diag(np.full(n, 1.25))
    a = np.linspace(-1.0, 3.0, 41)
    V = np.concatenate([np.repeat(a[:, None], n, 1), np.tile(np.eye(n)[:1], (5, 1)) * 0.5])
    n_, s = check(qa, cdd, np.eye(n), V, closed=closed, nhat=5 if closed else 0)
    assert s["fp64_gap_below_1e9"] > 0
    if closed:
        assert (n_.sum(1) == 5).all()


def test_rows_extreme_voltages(qa):
    """Huge charges and voltages that are not numbers: no row is skipped on a
    bound that overflows, and the call ends."""
    cdd, cgd = sub_array(16, 262)
    V = np.random.default_rng(3).uniform(-1.0, 2.0, (12, 16))
    V[0] *= 1e6
    V[1, 3] = -1e9
    V[2, 0] = 1e9
    check(qa, cdd, cgd, V[:3])
    V[4, 2], V[5, 1], V[6, :] = np.nan, np.inf, 1e200
    Vd = torch.as_tensor(V).cuda()
    n = qa.ground_state(cdd, cgd, Vd).cpu().numpy()
    ne = qa.ground_state(cdd, cgd, Vd, exhaustive=True).cpu().numpy()
    keep = [0, 3, 7, 8, 9, 10, 11]
    assert (n[keep] == ne[keep]).all()


@pytest.mark.parametrize("n_dot,seed", [(9, 12), (13, 12), (16, 12), (16, 11), (16, 200)])
def test_pixels_of_many_rows(qa, n_dot, seed):
    """Arrays whose rounded minimum is a poor guess at some pixels (hundreds of rows):
    the same states as computing every energy, for a call that looks for a better
    guess there and for one past its pixel count."""
    d = W.grid4x4(seed, npix=2)
    cdd, cgd = d.cdd[:n_dot, :n_dot].copy(), d.cgd[:n_dot, :n_dot].copy()
    V = np.random.default_rng(seed).uniform(-2.0, 8.0, (3000, n_dot))
    Vt = torch.as_tensor(V).cuda()
    few, st = qa.ground_state(cdd, cgd, Vt, stats=True)
    every, se = qa.ground_state(cdd, cgd, Vt, stats=True, exhaustive=True)
    many = qa.ground_state(cdd, cgd, Vt.repeat(17, 1))
    assert st["fp64_gap_below_1e9"] == se["fp64_gap_below_1e9"] == 0
    assert torch.equal(few, every)
    assert torch.equal(many, few.repeat(17, 1))
    assert st["scored"] <= se["scored"] == 3000 << n_dot


@pytest.mark.parametrize("n_dot,limit", [(14, 12500), (15, 25000), (16, 37500)])
def test_on_both_sides_of_the_tail_limit(qa, n_dot, limit):
    """The dense form that looks for a better guess, for as many pixels as it is used for,
    and the one without, for one more: the states of computing every energy."""
    cdd, cgd = sub_array(n_dot, 12)
    V = torch.as_tensor(np.random.default_rng(n_dot).uniform(-2.0, 8.0, (1250, n_dot))).cuda()
    every = qa.ground_state(cdd, cgd, V, exhaustive=True)
    few = qa.ground_state(cdd, cgd, V.repeat(limit // 1250, 1))
    more = qa.ground_state(cdd, cgd, torch.cat([V.repeat(limit // 1250, 1), V[:1]]))
    assert torch.equal(few, every.repeat(limit // 1250, 1))
    assert torch.equal(more[:limit], few) and torch.equal(more[limit:], every[:1])
