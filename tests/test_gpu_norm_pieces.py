"""Norms of a batch in which one LP has 1024 pieces and thousands have one."""
import numpy as np
import pytest

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
