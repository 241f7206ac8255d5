"""Sorted tiles (a choice of the tuner, pinned here through its cache file)
with adaptive steps, restarts to the average, a diagonal Hessian and finished
instances cut out of the launches: the products keep their places, so every
result has the bits of unsorted tiles of the same size.  And what the handle
reports of a layout."""
import os
import subprocess
import sys

import pytest

pytestmark = pytest.mark.gpu
ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

COMMON = """
import sys
sys.path[:0] = [%r, %r]
import numpy as np
from paper_2307_03466_amd import instances as I, pdhg
from test_gpu_edge import _lp_rows
BATCHES = [
    [_lp_rows([0] * 2050 + [1, 8192, 0, 4096, 4097, 3, 8193, 2, 9000], 20000, seed=1)],
    [_lp_rows([2] * 1025 + [0], 300, seed=3), _lp_rows([5, 4096, 1, 8191], 9000, seed=4), I.set_cover(30, 70, seed=5)],
    [I.set_cover(30, 70, seed=k) for k in range(40)] + [I.cover_knapsack(3000, seed=9)],
]
""" % (ROOT, os.path.join(ROOT, "tests"))

FIRST = COMMON + """
for lps in BATCHES:
    for prec in (0, 1):
        with pdhg.Batch(lps, precision=prec) as b:
            b.solve(tol=-1.0, iter_limit=8, fused_window=0)  # tunes, and writes its choice to the file
"""

OPTIONS = COMMON + """
OPTS = [dict(adaptive=1), dict(restart_avg=1), dict(adaptive=1, restart_avg=1), dict(quadratic=1),
        dict(tol=1e-2, compact=1), dict(tol=1e-2, compact=0), dict(tol=1e-2, compact=1, adaptive=1)]

def run(b, lps, quadratic=0, **kw):
    if quadratic:
        for q, lp in enumerate(lps):
            b.set_quadratic(q, 0.5 + np.arange(lp.n) % 3)
    res = b.solve(**{**dict(tol=-1.0, iter_limit=200, check_period=16, fused_window=0), **kw})
    return [(r["iterations"], r["status"]) for r in res], [b.solution(q) for q in range(len(lps))]

for lps in BATCHES:
    for prec in (0, 1):
        for kw in OPTS:
            out = []
            for chosen in (True, False):
                with pdhg.Batch(lps, precision=prec) as b:
                    if not chosen:
                        b.set_layout(0, -16, 0, -16)
                    out.append(run(b, lps, **kw))
                    info = b.info()
                    assert info["row_chunk"] == info["col_chunk"] == 4096, info
                    assert info["row_staged_variant"] == info["col_staged_variant"] == (4 if chosen else 0), info
            assert out[0][0] == out[1][0], (prec, kw)
            for (x0, y0), (x1, y1) in zip(out[0][1], out[1][1]):
                assert np.array_equal(x0, x1) and np.array_equal(y0, y1), (prec, kw)
print("options ok")
"""

# ept, flags, blocks of both orientations -> chunk, variant, plain loads in FP64 and FP32
REPORT = COMMON + """
chunk, variant, plain64, plain32 = map(int, sys.argv[1:5])
lps = BATCHES[0]
for prec, plain in ((pdhg.FP64, plain64), (pdhg.FP32, plain32)):
    with pdhg.Batch(lps, precision=prec) as b:
        b.solve(tol=-1.0, iter_limit=8, fused_window=0)
        info = b.info()
        for d in ("row", "col"):
            assert info[d + "_chunk"] == chunk and info[d + "_staged_variant"] == variant, info
            assert info[d + "_cached"] == plain, info
print("report ok")
"""


def _run(code, path, *args):
    env = dict(os.environ, SCYLLA_TUNE_CACHE=str(path), SCYLLA_CUT_TRACE="1")
    return subprocess.run([sys.executable, "-c", code, *args], env=env, capture_output=True, text=True, timeout=110)


@pytest.fixture(scope="module")
def keys(tmp_path_factory):
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    path = tmp_path_factory.mktemp("tune") / "first.txt"
    r = _run(FIRST, path)
    assert r.returncode == 0, r.stderr[-2000:]
    return [line.split()[0] for line in path.read_text().splitlines()]


@pytest.mark.parametrize("flags", [128, 192])
def test_options_over_sorted_tiles(keys, tmp_path, flags):
    path = tmp_path / "second.txt"
    path.write_text("".join(f"{k} 0 -16 0 {flags} 0 -16 0 {flags}\n" for k in keys))
    r = _run(OPTIONS, path)
    assert r.returncode == 0 and "options ok" in r.stdout, r.stdout[-500:] + r.stderr[-2000:]
    assert "cut after window" in r.stderr


@pytest.mark.parametrize("blocks,ept,flags,chunk,variant,plain64,plain32",
                         [(0, -32, 192, 8192, 4, 1, 1), (0, -16, 128, 4096, 4, 0, 0), (0, 8, 64, 2048, 0, 1, 1),
                          (2, 8, 64, 2048, 0, 0, 1), (2, 4, 0, 1024, 0, 0, 0)])
def test_reported_layout(keys, tmp_path, blocks, ept, flags, chunk, variant, plain64, plain32):
    path = tmp_path / "report.txt"
    path.write_text("".join(f"{k} {blocks} {ept} 0 {flags} {blocks} {ept} 0 {flags}\n" for k in keys))
    r = _run(REPORT, path, *map(str, (chunk, variant, plain64, plain32)))
    assert r.returncode == 0 and "report ok" in r.stdout, r.stdout[-500:] + r.stderr[-2000:]
