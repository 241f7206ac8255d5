"""Device fix-and-propagate where its lane groups change: rows of 15 to 33
nonzeros (16 lanes a row), columns of 7 to 17 (8 lanes a column), more
selections a batch than threads (1024); bit for bit the oracle's."""
import numpy as np
import pytest

import oracle
from lp_util import lp_from_dense

pytestmark = pytest.mark.gpu
pdhg = pytest.importorskip("paper_2307_03466_amd.pdhg")


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    torch.cuda.set_device(0)
    pdhg.lib()


def _lp(rows, n, seed, unbounded):
    """Rows of the given lengths over n columns, mixed senses and signs, fractional
    coefficients (sums that round), explicit zeros, a few infinite bounds."""
    rng = np.random.default_rng(seed)
    A = np.zeros((len(rows), n))
    for i, k in enumerate(rows):
        j = rng.choice(n, size=k, replace=False)
        A[i, j] = rng.integers(-9, 10, size=k) / 7.0
    x = rng.integers(0, 3, size=n).astype(float)
    ax = A @ x
    senses = "".join(rng.choice(list("GLE"), size=len(rows), p=[0.45, 0.45, 0.1]))
    b = ax + np.where(np.array(list(senses)) == "G", -1.0, np.where(np.array(list(senses)) == "L", 1.0, 0.0)) * rng.random(len(rows))
    l, u = np.zeros(n), np.full(n, 3.0)
    if unbounded:
        u[rng.random(n) < 0.2] = np.inf
        l[rng.random(n) < 0.1] = -np.inf
    lp = lp_from_dense(A, b, senses, rng.normal(size=n), l, u)
    lp.is_int = (rng.random(n) < 0.8).astype(np.uint8)
    return lp, np.clip(x + rng.normal(scale=0.4, size=n), np.maximum(l, -4), np.minimum(u, 4))


@pytest.mark.parametrize("K", [1, 7, 1023, 1024, 1025])
@pytest.mark.parametrize("unbounded", [False, True])
def test_lane_groups_at_their_limits(K, unbounded):
    cases = [_lp([15, 16, 17, 31, 32, 33, 1, 0, 16], 40, 1, unbounded),
             _lp([5] * 60, 24, 2, unbounded),           # columns of about 12 rows
             _lp([3] * 700, 1500, 3, unbounded)]        # more columns than threads
    lps, xs = [c[0] for c in cases], [c[1] for c in cases]
    with pdhg.Batch(lps) as b:
        xh, feas, ign, mask = b.fix_propagate(K, is_int=np.concatenate([lp.is_int for lp in lps]),
                                              xbar=np.concatenate(xs))
    c0 = r0 = 0
    for q, (lp, x) in enumerate(zip(lps, xs)):
        ex, eok, en, emask = oracle.fix_propagate_batched(lp, x, K=K)
        assert np.array_equal(xh[c0:c0 + lp.n], ex) and feas[q] == eok and ign[q] == en
        assert np.array_equal(mask[r0:r0 + lp.m], emask)
        c0, r0 = c0 + lp.n, r0 + lp.m
