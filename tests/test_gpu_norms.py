"""Norms and cold-start weight of an instance, at the edges of the pieces
they are summed in (8192 entries a piece, at most 256 pieces), after setup
and after one instance of a batch got a new objective."""
import numpy as np
import pytest

import oracle
from paper_2307_03466_amd import instances as I

pytestmark = pytest.mark.gpu
pdhg = pytest.importorskip("paper_2307_03466_amd.pdhg")

M = 90


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    torch.cuda.set_device(0)
    pdhg.lib()


def _lp(n, seed):
    """M rows of three columns each, spread over all n columns."""
    rng = np.random.default_rng(seed)
    col = np.sort((np.arange(3 * M) * (n // (3 * M)) + n % (3 * M)).reshape(M, 3), axis=1)
    return I.LP(m=M, n=n, row_ptr=np.arange(0, 3 * M + 1, 3), col_idx=col.ravel().astype(np.int32),
                val=rng.integers(1, 9, size=3 * M).astype(float), c=rng.normal(size=n), b=rng.normal(size=M),
                senses=np.full(M, ord("G"), dtype=np.uint8), l=np.zeros(n), u=np.ones(n),
                is_int=np.zeros(n, dtype=np.uint8))


def _expect(lp, c):
    dr, dc = oracle.precondition(lp)[:2]
    omega = np.linalg.norm(dc * c) / np.linalg.norm(dr * lp.b)
    return omega, oracle.kkt(lp, np.zeros(lp.n), np.zeros(lp.m), c=c)["rel"]


@pytest.mark.parametrize("total", [M + 270, 8191, 8192, 8193, 16385, 2_097_153, 2_200_001])
def test_norms_at_piece_edges(total):
    lps = [_lp(500, 1), _lp(total - M, 2), _lp(8193 - M, 3)]
    c2 = np.random.default_rng(4).normal(size=lps[1].n) * 3.0
    # an FP64 sum of N terms is off by at most N eps
    tol = 2 * total * np.finfo(float).eps + 1e-12
    with pdhg.Batch(lps, precision=pdhg.FP64) as b:
        for objs in ([lp.c for lp in lps], [lps[0].c, c2, lps[2].c]):
            b.set_objective(1, objs[1])
            for q, r in enumerate(b.solve(tol=1e-300, iter_limit=0, autotune=0)):
                omega, rel = _expect(lps[q], objs[q])
                assert r["iterations"] == 0
                assert abs(r["omega"] - omega) <= tol * omega
                assert abs(r["rel_kkt"] - rel) <= tol * rel
