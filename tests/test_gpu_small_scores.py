"""Ground states of 1..8 dots, which the setup kernel scores itself: groups of 2, 4
and 8 lanes with and without idle dots, dense and thresholded sets, open and closed,
at pixel counts around a block of 448 lanes; integer states are compared exactly away
from ties (a gap below 1e-9), the statistics with the sets' sizes."""
import math

import numpy as np
import pytest
import torch

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


@pytest.mark.parametrize("closed,t", [(False, 1.0), (False, 0.4), (True, 1.0), (True, 0.3)])
@pytest.mark.parametrize("n", range(1, 9))
def test_small_scores(qa, oracle, n, closed, t):
    rng = np.random.default_rng(800 + n)
    cdd = np.diag(rng.uniform(1.0, 1.4, n))
    for i in range(n - 1):
        cdd[i, i + 1] = cdd[i + 1, i] = -rng.uniform(0.1, 0.3)
    cgd = np.diag(rng.uniform(0.5, 1.0, n)) + rng.uniform(0.0, 0.1, (n, n))
    group = 2 if n <= 2 else (4 if n <= 4 else 8)
    kw = dict(closed=closed, nhat=n if closed else 0, t=t)
    for pixels in (1, 448 // group - 1, 448 // group, 448 // group + 1, 1500):
        V = rng.uniform(-1.5, 4.0, (pixels, n))
        print(n, pixels, kw, flush=True)
        got, st = qa.ground_state(cdd, cgd, torch.as_tensor(V).cuda(), stats=True, **kw)
        ref = oracle.method_gs(cdd, cgd, V, **kw)
        gap = ref["e2"] - ref["e1"]
        clear = (gap > 1e-9) & ((ref["info"] & oracle.INFO_AMBIGUOUS) == 0)
        assert (got.cpu().numpy() == ref["n"])[clear].all()
        if closed:
            assert (got.cpu().numpy().sum(1) == n).all()
        assert st["pixels"] == pixels and st["qp_failures"] == 0
        free = np.array([bin(int(m)).count("1") for m in ref["freemask"]]) if "freemask" in ref else None
        if t == 1.0 and not closed:
            assert st["candidates"] == pixels << n
        elif free is not None:
            assert st["candidates"] == sum(
                math.comb(int(f), int(k)) if closed else 1 << int(f) for f, k in zip(free, ref["k"]))


def test_not_a_number(qa):
    """A voltage that is not a number leaves the other pixels as they are."""
    cdd = np.diag([1.2, 1.1, 1.3])
    cgd = np.diag([0.7, 0.8, 0.9])
    V = torch.linspace(0.0, 3.0, 300, dtype=torch.float64).reshape(100, 3).cuda()
    want = qa.ground_state(cdd, cgd, V)
    V[7, 1] = float("nan")
    got = qa.ground_state(cdd, cgd, V)
    keep = torch.arange(100, device="cuda") != 7
    assert torch.equal(got[keep], want[keep])
