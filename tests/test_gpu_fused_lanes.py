"""The fused window keeps a row's entries in the registers of its lanes (8 a
lane in FP64, 16 in FP32, up to 64 lanes a row) when there is at most one row
or column a thread, and reads them from LDS otherwise: both sides of each
limit against the oracle."""
import pytest

import oracle
from lp_util import parity_err
from test_gpu_edge import _lp_rows

pytestmark = pytest.mark.gpu
pdhg = pytest.importorskip("paper_2307_03466_amd.pdhg")


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    torch.cuda.set_device(0)
    pdhg.lib()


# 16 rows: 64 lanes a row, 512 (FP64) or 1024 (FP32) entries in registers;
# 33 rows: 16 lanes, 128 or 256 entries; 1025 columns: beyond one a thread
@pytest.mark.parametrize("prec,lengths,n", [
    (0, [511, 3, 0, 512], 600), (0, [513, 1], 600), (0, [128] + [2] * 32, 300), (0, [129] + [2] * 32, 300),
    (0, [5] * 9, 1024), (0, [5] * 9, 1025), (0, [1], 1),
    (1, [1024, 7], 1024), (1, [1023, 0, 900], 1025), (1, [256] + [3] * 32, 400), (1, [257] + [3] * 32, 400),
    (1, [1] * 1024, 40), (1, [1] * 1025, 40)])
@pytest.mark.parametrize("adaptive", [0, 1])
def test_lanes_at_their_limits(prec, lengths, n, adaptive):
    lp = _lp_rows(lengths, n, seed=len(lengths) + n)
    # the repository's bounds: 100 fixed steps, or 30 (FP64) / 10 (FP32) adaptive ones
    iters = (30 if prec == 0 else 10) if adaptive else 100
    ref = oracle.pdhg(lp, tol=-1.0, iter_limit=iters, restarts=False, **({"adaptive": True} if adaptive else {}))
    with pdhg.Batch([lp], precision=prec) as b:
        assert b.info()["fused_eligible"] == 1
        r = b.solve(tol=-1.0, iter_limit=iters, restarts=0, adaptive=adaptive, autotune=0)[0]
        x, y = b.solution(0)
        rerun = b.solve(tol=-1.0, iter_limit=iters, restarts=0, adaptive=adaptive, autotune=0)[0]
        x2, y2 = b.solution(0)
    assert r["iterations"] == rerun["iterations"] == iters
    assert (x == x2).all() and (y == y2).all()
    bar = 1e-10 if prec == 0 else (1e-3 if adaptive else 1e-4)
    assert parity_err(x, y, ref.x, ref.y) <= bar
