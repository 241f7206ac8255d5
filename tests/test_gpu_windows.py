"""Where a solve's launches change with its iteration limit: whole windows of
64 iterations as a graph, a short last window launched by itself (up to half
of one) or as a graph (more than half), no iterations behind the last check;
and the launches of the fused form, 4096 iterations each."""
import pytest

import oracle
from paper_2307_03466_amd import instances as I
from lp_util import parity_err

pytestmark = pytest.mark.gpu
pdhg = pytest.importorskip("paper_2307_03466_amd.pdhg")


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    torch.cuda.set_device(0)
    pdhg.lib()


def _check(lp, limit, fused):
    ref = oracle.pdhg(lp, tol=-1.0, iter_limit=limit, restarts=False)
    with pdhg.Batch([lp], precision=pdhg.FP64) as b:
        for _ in range(2):  # the second solve reuses what the first one made
            r = b.solve(tol=1e-300, iter_limit=limit, restarts=0, fused_window=fused, autotune=0)[0]
            assert r["iterations"] == limit and r["status"] == pdhg.ITERATION_LIMIT
            # fixed-iteration parity of the FP64 path
            assert parity_err(*b.solution(0), ref.x, ref.y) <= 1e-10


@pytest.mark.parametrize("fused", [0, 1])
@pytest.mark.parametrize("limit", [0, 1, 32, 33, 63, 64, 65, 96, 97, 129])
def test_limits_around_windows(limit, fused):
    _check(I.set_cover(40, 100, seed=5), limit, fused)


@pytest.mark.parametrize("limit", [4095, 4096, 4097, 4161])
def test_limits_around_fused_launches(limit):
    _check(I.set_cover(30, 70, seed=6), limit, 1)


@pytest.mark.parametrize("fused", [0, 1])
def test_largest_iteration_limit(fused):
    """No limit, as large as the parameter holds: ends at its tolerance."""
    lp = I.set_cover(30, 70, seed=6)
    with pdhg.Batch([lp], precision=pdhg.FP64) as b:
        r = b.solve(tol=1e-4, iter_limit=2**63 - 1, fused_window=fused, autotune=0)[0]
        x, y = b.solution(0)
    assert r["status"] == pdhg.OPTIMAL and oracle.kkt(lp, x, y)["rel"] <= 1e-4 * (1 + 1e-6)
