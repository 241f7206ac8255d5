"""Norms of a batch in which one LP has 1024 pieces and thousands have one."""
import numpy as np
import pytest

from paper_2307_03466_amd import instances as I
from test_gpu_norms import M, _expect, _lp

pytestmark = pytest.mark.gpu
pdhg = pytest.importorskip("paper_2307_03466_amd.pdhg")


@pytest.mark.parametrize("before,after", [(0, 3), (16384, 0), (9000, 8000)])
def test_one_large_lp_among_many_small_ones(before, after):
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    kinds = [_lp(300, 1), _lp(5000 - M, 2), _lp(2_150_000, 3)]
    which = [k % 2 for k in range(before)] + [2] + [k % 2 for k in range(after)]
    c = [lp.c for lp in kinds] + [np.random.default_rng(4).normal(size=kinds[2].n) * 3.0]
    # an FP64 sum of N terms is off by at most N eps
    tol = [2 * (lp.n + M) * np.finfo(float).eps + 1e-12 for lp in kinds]
    with pdhg.Batch([kinds[k] for k in which], precision=pdhg.FP64) as b:
        for big in (2, 3):
            b.set_objective(before, c[big])
            want = [_expect(kinds[k], c[big if k == 2 else k]) for k in range(3)]
            for k, r in zip(which, b.solve(tol=1e-300, iter_limit=0, autotune=0)):
                assert abs(r["omega"] - want[k][0]) <= tol[k] * want[k][0]
                assert abs(r["rel_kkt"] - want[k][1]) <= tol[k] * want[k][1]


def test_ranges_of_instances():
    """The L2 loop refreshes the norms of one group of instances at a time:
    two groups, of instances with different numbers of pieces, give the
    results of one."""
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    lps = [I.cover_knapsack(m, seed=m) for m in (2500, 300, 700, 5200, 400, 1500)]
    out = []
    with pdhg.Batch(lps) as b:
        b.set_layout(0, 4, 0, 4)
        for pipeline in (0, 1):
            recs, fin, x = b.pump_ex(pump=dict(rounds=4, early_exit=0, distance=2, pipeline=pipeline), iter_limit=640)
            out.append(([[(r["iterations"], r["rel_kkt"], r["xhat_obj"]) for r in k] for k in recs], x))
    assert out[0][0] == out[1][0]
    assert np.array_equal(out[0][1], out[1][1])
