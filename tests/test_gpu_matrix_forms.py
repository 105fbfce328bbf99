"""The matrix-core scorers themselves: computing every energy (exhaustive) for 9..16 dots,
all set families and precisions, against the FP64 oracle; and the bound-ordered search
on both sides of the pixel counts from which FP64 rows take its place."""
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


def diagram(n_dot):
    """A chain with next-nearest couplings; half of the pixels within some 1e-8 of a charge
    transition (near ties for every approximate form): with x_u = n + e_i / 2 + C_dd w the
    states n and n + e_i differ by w_i in energy."""
    rng = np.random.default_rng(90 + n_dot)
    cdd = np.diag(rng.uniform(1.0, 1.4, n_dot))
    for k, lo, hi in ((1, 0.1, 0.3), (2, 0.02, 0.06)):
        for i in range(n_dot - k):
            cdd[i, i + k] = cdd[i + k, i] = -rng.uniform(lo, hi)
    cgd = np.diag(rng.uniform(0.5, 1.0, n_dot))
    x = rng.uniform(-0.5, 3.5, (400, n_dot))
    p, i = np.arange(200), rng.integers(0, n_dot, 200)
    w = rng.uniform(-0.1, 0.1, (200, n_dot))
    w[p, i] = 1e-8 * rng.standard_normal(200)
    x[:200] = rng.integers(1, 4, (200, n_dot)) + w @ cdd
    x[p, i] += 0.5
    return W.Diagram(cdd, cgd, np.linalg.solve(cgd, x.T).T.copy())


@pytest.mark.parametrize("prec", ["fp32", "bf16x3", "bf16x2"])
@pytest.mark.parametrize("closed,t", [(False, 1.0), (False, 0.6), (True, 1.0), (True, 0.5)])
@pytest.mark.parametrize("n_dot", [9, 10, 11, 12, 13, 14, 15, 16])
def test_every_energy(qa, oracle, n_dot, closed, t, prec):
    d = diagram(n_dot)
    kw = dict(closed=closed, nhat=n_dot if closed else 0, t=t)
    n, st = qa.ground_state(d.cdd, d.cgd, torch.as_tensor(d.V).cuda(), precision=prec,
                            exhaustive=True, stats=True, **kw)
    n = n.cpu().numpy()
    ref = oracle.method_gs(d.cdd, d.cgd, d.V, **kw)
    excl = (ref["e2"] - ref["e1"] < 1e-9) | ((ref["info"] & oracle.INFO_AMBIGUOUS) > 0)
    assert ((n == ref["n"]).all(1) | excl).all()
    assert excl.sum() < 40
    assert st["candidates"] == st["scored"] == (400 << n_dot if t == 1.0 and not closed
                                                else ref["ncand"].sum())
    # what the matrix cores leave to the FP64 re-score (the FP64 forms have none)
    if not closed and t == 1.0:
        assert st["near_tie_pixels"] > 0


@pytest.mark.parametrize("prec", ["bf16x3", "bf16x2"])
@pytest.mark.parametrize("n_dot,t,limit", [(15, 1.0, 24000), (16, 1.0, 48000), (16, 0.5, 16000)])
def test_both_sides_of_the_limit(qa, n_dot, t, limit, prec):
    d = W.grid4x4(290, npix=2)
    cdd, cgd = d.cdd[:n_dot, :n_dot].copy(), d.cgd[:n_dot, :n_dot].copy()
    V = torch.as_tensor(np.random.default_rng(limit).uniform(-1.0, 3.0, (limit + 1, n_dot))).cuda()
    rows, sr = qa.ground_state(cdd, cgd, V, t=t, stats=True)
    few, sf = qa.ground_state(cdd, cgd, V[:limit], t=t, precision=prec, stats=True)
    many, sm = qa.ground_state(cdd, cgd, V, t=t, precision=prec, stats=True)
    assert sf["near_tie_pixels"] > 0 == sm["near_tie_pixels"]  # which scorer ran
    diff = int((few != rows[:limit]).any(1).sum())
    assert diff <= sr["fp64_gap_below_1e9"] and torch.equal(many, rows)
    assert sm["candidates"] == sr["candidates"] and sf["scored"] < sf["candidates"] or t < 1.0


@pytest.mark.parametrize("prec", ["bf16x3", "bf16x2"])
@pytest.mark.parametrize("t", [0.0, 0.3, 0.6, 0.9])
def test_thresholded_bound_order(qa, oracle, t, prec):
    """Bound-ordered search of the thresholded sub-boxes against the oracle, random
    capacitances and an array."""
    for d in (W.paper_replica(16, seed=740, npix=20), W.grid4x4(291, npix=20)):
        n, st = qa.ground_state(d.cdd, d.cgd, torch.as_tensor(d.V).cuda(), t=t, precision=prec,
                                stats=True)
        ref = oracle.method_gs(d.cdd, d.cgd, d.V, t=t)
        excl = (ref["e2"] - ref["e1"] < 1e-9) | ((ref["info"] & oracle.INFO_AMBIGUOUS) > 0)
        assert ((n.cpu().numpy() == ref["n"]).all(1) | excl).all()
        assert st["candidates"] == ref["ncand"].sum()
