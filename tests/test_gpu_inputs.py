"""The inputs of a single-diagram call as arguments of the setup kernel (up to 440
doubles: a triangle of C_dd, C_gd and a sweep) or by a copy into the record: sizes
on both sides of the limit, problems in turn on one stream, and the calls that read
the record afterwards.  Integer ground states are compared exactly away from ties
(a gap below 1e-9)."""
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


@pytest.fixture(scope="module")
def oracle():
    import oracle as O
    O.build()
    return O


def problem(n, g, seed):
    rng = np.random.default_rng(seed)
    cdd = np.diag(rng.uniform(1.0, 1.4, n))
    for i in range(n - 1):
        cdd[i, i + 1] = cdd[i + 1, i] = -rng.uniform(0.1, 0.3)
    return cdd, rng.uniform(0.0, 0.4, (n, g)), rng


@pytest.mark.parametrize("n,g", [(1, 1), (2, 32), (3, 5), (8, 32), (12, 30), (12, 31), (16, 16),
                                 (16, 17), (16, 19), (16, 20), (16, 32)])
def test_arguments_and_record(qa, oracle, n, g):
    cdd, cgd, rng = problem(n, g, 500 + 40 * n + g)
    bent = cdd.copy()
    if n > 1:
        bent[0, 1] = np.nextafter(bent[0, 1], 0.0)  # symmetric to rounding only: copied
    V = rng.uniform(-1.0, 4.0, (37, g))
    Vt = torch.as_tensor(V).cuda()
    for closed in (False, True):
        kw = dict(closed=closed, nhat=n if closed else 0)
        ref = oracle.method_gs(cdd, cgd, V, **kw)
        clear = ref["e2"] - ref["e1"] > 1e-9
        for c in (cdd, bent, cdd):
            print(n, g, closed, c is bent, flush=True)
            got = qa.ground_state(c, cgd, Vt, **kw).cpu().numpy()
            assert (got == ref["n"])[clear].all()
        other = qa.ground_state(cdd, 0.5 * cgd, Vt, **kw).cpu().numpy()
        ref2 = oracle.method_gs(cdd, 0.5 * cgd, V, **kw)
        assert (other == ref2["n"])[ref2["e2"] - ref2["e1"] > 1e-9].all()
        out = torch.empty((37, n), dtype=torch.int32, device="cuda")
        qa.ground_state_noalloc(cdd, cgd, Vt, out, **kw)
        assert (out.cpu().numpy() == ref["n"])[clear].all()
        # a sweep, its arguments fewer gates
        y = rng.uniform(0.0, 1.0, (3, g))
        sweep = dict(v0=y[0], e1=y[1], e2=y[2], a0=-1.0, a1=3.0, nx=7, b0=0.0, b1=2.0, ny=5)
        Vs = torch.as_tensor(W.sweep_voltages(sweep)).cuda()
        a = qa.ground_state_grid(cdd, cgd, sweep, **kw)
        assert torch.equal(a.view(35, n), qa.ground_state(cdd, cgd, Vs, **kw))


@pytest.mark.parametrize("n", [2, 8, 12])
def test_adjoint_after_arguments(qa, oracle, n):
    """The adjoint reads the record that a forward call stored from its arguments."""
    cdd, cgd, rng = problem(n, n + 1, 700 + n)
    V = rng.uniform(-1.0, 4.0, (33, n + 1))
    Gb = rng.standard_normal((33, n))
    st = oracle.method_setup(cdd, cgd, V)
    want = oracle.soft_grad(cdd, cgd, V, 0.05, st["n0"], st["freemask"], st["k"], Gb)
    Vt, Gt = torch.as_tensor(V).cuda(), torch.as_tensor(Gb).cuda()
    qa.ground_state(2.0 * cdd, cgd, Vt)
    _, saved = qa.soft_charge(cdd, cgd, Vt, 0.05)
    got = qa.soft_charge_backward(cdd, cgd, Vt, 0.05, Gt, saved)
    for a, b in zip(got, want):
        assert np.linalg.norm(a.cpu().numpy() - b) <= 1e-9 * max(np.linalg.norm(b), 1e-300)
