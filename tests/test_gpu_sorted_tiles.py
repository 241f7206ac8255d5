"""Normal tiles with their entries sorted by what they gather (4096 or 8192
nonzeros), and those of 256 nonzeros: pinned through the tuning cache file, since the layout call offers
the unsorted ones only.  The products keep their places, so 4096-nonzero
sorted tiles give the unsorted ones' bits; both are checked against the
oracle, at tile edges, with long rows, empty rows, one instance and a batch,
and the passes of a choice that a file cannot hold stay in bounds."""
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
rng = np.random.default_rng(3)
BATCHES = [
    [_lp_rows([0] * 2050 + [1, 8192, 0, 4096, 4097, 3, 8193, 2, 9000], 20000, seed=1)],
    [_lp_rows([3] * 3000, 700, seed=2)],
    [_lp_rows([2] * 1025 + [0], 300, seed=3), _lp_rows([5, 4096, 1, 8191], 9000, seed=4), I.set_cover(30, 70, seed=5)],
]
KW = dict(tol=-1.0, iter_limit=100, restarts=0, fused_window=0)
""" % (ROOT, os.path.join(ROOT, "tests"))

FIRST = COMMON + """
for lps in BATCHES:
    for prec in (0, 1):
        with pdhg.Batch(lps, precision=prec) as b:
            b.solve(**KW)  # tunes, and writes its choice to the file
"""

SECOND = COMMON + """
import oracle
from lp_util import parity_err
want = int(sys.argv[1])
for lps in BATCHES:
    refs = [oracle.pdhg(lp, tol=-1.0, iter_limit=100, restarts=False) for lp in lps]
    for prec in (0, 1):
        with pdhg.Batch(lps, precision=prec) as b:
            b.solve(**KW)
            info = b.info()
            chunk = {-32: 8192, 1: 256}.get(want, 4096)
            assert info["row_chunk"] == info["col_chunk"] == chunk, info
            got = [b.solution(q) for q in range(len(lps))]
        for q in range(len(lps)):
            assert parity_err(*got[q], refs[q].x, refs[q].y) <= (1e-10 if prec == 0 else 1e-4)
        if chunk == 4096:
            with pdhg.Batch(lps, precision=prec) as b:
                b.set_layout(0, -16, 0, -16)
                b.solve(**KW)
                for q in range(len(lps)):
                    x, y = b.solution(q)
                    assert np.array_equal(x, got[q][0]) and np.array_equal(y, got[q][1])
print("sorted ok")
"""


def _run(code, path, *args):
    env = dict(os.environ, SCYLLA_TUNE_CACHE=str(path))
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


# ept, flags of a sorted choice (128), with plain loads (64); -32 without the
# flag is no choice: its passes run 4096-nonzero tiles; 1: the 256-nonzero
# tiles of small LPs, which the layout call does not offer either
@pytest.mark.parametrize("ept,flags,want", [(-16, 128, -16), (-32, 128, -32), (-16, 192, -16), (-32, 192, -32),
                                            (-32, 0, -16), (1, 0, 1), (1, 64, 1)])
def test_sorted_tiles(keys, tmp_path, ept, flags, want):
    path = tmp_path / "second.txt"
    path.write_text("".join(f"{k} 0 {ept} 0 {flags} 0 {ept} 0 {flags}\n" for k in keys))
    r = _run(SECOND, path, str(want))
    assert r.returncode == 0 and "sorted ok" in r.stdout, r.stdout[-500:] + r.stderr[-2000:]
