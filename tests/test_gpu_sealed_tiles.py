"""Normal tiles carry their nonzero range: tiles at the row and nonzero limits
of every tile size, empty rows at the ends, segments of long rows, for one
instance (entries loaded before the state) and for a batch (after it)."""
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


@pytest.mark.parametrize("ept", [2, 4, 8, 16, -8, -16])
@pytest.mark.parametrize("prec", [0, 1])
def test_tiles_at_their_limits(ept, prec):
    chunk = 256 * abs(ept)
    lps = [_lp_rows([0] * 1030 + [1, chunk, 0, chunk + 1, 3, chunk - 1, 2, 2 * chunk], 2 * chunk + 5, seed=ept + 20),
           _lp_rows([1] * 1025 + [0], 300, seed=ept + 40)]
    refs = [oracle.pdhg(lp, tol=-1.0, iter_limit=100, restarts=False) for lp in lps]
    bar = 1e-10 if prec == 0 else 1e-4  # fixed-iteration parity of each path
    for part in ([0], [1], [0, 1]):
        with pdhg.Batch([lps[q] for q in part], precision=prec) as b:
            b.set_layout(0, ept, 0, ept)
            b.solve(tol=-1.0, iter_limit=100, restarts=0, fused_window=0, autotune=0)
            for k, q in enumerate(part):
                assert parity_err(*b.solution(k), refs[q].x, refs[q].y) <= bar


# step-size partials of about 980 and 3910 tiles: beyond one turn of the 960
# summing threads, and beyond one round of four turns
@pytest.mark.parametrize("m", [50_000, 200_000])
def test_step_sums_beyond_a_round(m):
    from paper_2307_03466_amd import instances as I
    lp = I.general_lp(m, 2 * m, seed=m)
    ref = oracle.pdhg(lp, tol=-1.0, iter_limit=3, restarts=False, adaptive=True)
    with pdhg.Batch([lp], precision=0) as b:
        b.set_layout(0, 2, 0, 2)
        b.solve(tol=-1.0, iter_limit=3, restarts=0, adaptive=1, autotune=0)
        x, y = b.solution(0)
        b.solve(tol=-1.0, iter_limit=3, restarts=0, adaptive=1, autotune=0)
        x2, y2 = b.solution(0)
    assert parity_err(x, y, ref.x, ref.y) <= 1e-10  # the sums of the first steps, before they amplify rounding
    assert (x == x2).all() and (y == y2).all()
