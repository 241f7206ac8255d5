"""Norms and cold-start weight of an instance, at the edges of the pieces
they are summed in (2048 entries a piece, at most 1024 pieces), after setup
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


@pytest.mark.parametrize("total", [M + 270, 2047, 2048, 2049, 8193, 2_097_153, 2_200_001])
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


@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("total", [2048, 2049, 5000])
def test_blended_objective_at_piece_edges(prec, total):
    """The pump's objective and its norms are made in one pass over a piece;
    bits that end inside a byte, with and without continuous columns."""
    lps = [_lp(500, 1), _lp(total - M, 2), _lp(1000, 3)]
    lp = lps[1]
    rng = np.random.default_rng(5)
    up, ii = rng.random(lp.n) < 0.4, rng.random(lp.n) < 0.7
    a, kappa = 0.81, 1.7
    tol = 2 * total * np.finfo(float).eps + 1e-12
    with pdhg.Batch(lps, precision=prec) as b:
        for flags in (None, ii):
            b.set_blend(1, up, a, kappa, is_int=flags)
            c = a * kappa * lp.c + (1.0 - a) * np.where(ii if flags is not None else True, np.where(up, -1.0, 1.0), 0.0)
            for q, r in enumerate(b.solve(tol=1e-300, iter_limit=0, autotune=0)):
                omega, rel = _expect(lps[q], c if q == 1 else lps[q].c)
                assert abs(r["omega"] - omega) <= tol * omega
                assert abs(r["rel_kkt"] - rel) <= tol * rel


@pytest.mark.parametrize("m", [1, 15, 16, 17, 33, 4096, 4101])
def test_feasibility_flags_at_word_edges(m):
    """One violated row or column anywhere must show: the flags are read in
    words of 16 that need not start where an instance does."""
    def lp(m, bad):
        x = np.ones(m)
        b = np.ones(m)
        if bad is not None:
            b[bad] = 2.0  # row bad: x_bad >= 2, bounds hold x at 1
        return I.LP(m=m, n=m, row_ptr=np.arange(m + 1), col_idx=np.arange(m, dtype=np.int32), val=np.ones(m),
                    c=np.ones(m), b=b, senses=np.full(m, ord("G"), dtype=np.uint8), l=np.ones(m), u=x,
                    is_int=np.ones(m, dtype=np.uint8))
    at = sorted({0, m // 2, m - 1, max(0, m - 2), min(m - 1, 15), min(m - 1, 16)})
    lps = [lp(m, None)] + [v for k in at for v in (lp(m, k), lp(m, None))]
    with pdhg.Batch(lps) as b:
        b.solve(tol=-1.0, iter_limit=0, autotune=0)  # x = proj(0) = 1
        want = [1] + [v for _ in at for v in (0, 1)]
        assert b.mip_feasible().tolist() == want
        assert b.mip_feasible(is_int=np.zeros(m * len(lps), dtype=np.uint8)).tolist() == want


def test_updates_beyond_the_staging_buffer():
    """Updates are staged in a 1 MiB buffer that starts over once the stream
    has drained; larger ones are copied directly.  The last value of every
    instance counts, whatever was staged around it."""
    rng = np.random.default_rng(6)
    lps = [_lp(5000, 1), _lp(140_000, 2), _lp(700, 3)]
    with pdhg.Batch(lps, precision=pdhg.FP64) as b:
        want = [None] * 3
        for k in range(60):  # 60 x 40 KB
            for q in ([0, 2] if k else [0, 1, 2]):
                want[q] = rng.normal(size=lps[q].n)  # instance 1: 1.1 MB
                b.set_objective(q, want[q])
                want[q] = want[q].copy()
        for q, r in enumerate(b.solve(tol=1e-300, iter_limit=0, autotune=0)):
            omega, rel = _expect(lps[q], want[q])
            assert abs(r["omega"] - omega) <= 1e-9 * omega and abs(r["rel_kkt"] - rel) <= 1e-9 * rel
        a, kappa = 0.5, 2.0
        for k in range(120):  # 120 x 2 x (0.6 + 0.1) KB in place, 17.5 KB bits copied
            for q in ([0, 2] if k % 40 else [0, 1, 2]):
                up, ii = rng.random(lps[q].n) < 0.5, rng.random(lps[q].n) < 0.5
                b.set_blend(q, up, a, kappa, is_int=ii)
                want[q] = a * kappa * lps[q].c + (1 - a) * np.where(ii, np.where(up, -1.0, 1.0), 0.0)
        for q, r in enumerate(b.solve(tol=1e-300, iter_limit=0, autotune=0)):
            omega, rel = _expect(lps[q], want[q])
            assert abs(r["omega"] - omega) <= 1e-9 * omega and abs(r["rel_kkt"] - rel) <= 1e-9 * rel
