"""Updates staged around the place where the pinned staging buffer (1 MiB)
starts over, on a stream that is behind."""
import numpy as np
import pytest

from paper_2307_03466_amd import instances as I
from test_gpu_norms import _expect, _lp

pytestmark = pytest.mark.gpu
pdhg = pytest.importorskip("paper_2307_03466_amd.pdhg")


# objectives of 5100 columns (41 KB) staged first, so that of the bits of the
# next update (2 x 15 KB) both fit, or only the first
@pytest.mark.parametrize("first", [24, 25])
def test_bits_where_the_buffer_starts_over(first):
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    rng = np.random.default_rng(first)
    lps = [_lp(120_000, 1), _lp(129_000, 2), _lp(5100, 3)]
    stream = torch.cuda.Stream()
    up, ii = rng.random(lps[0].n) < 0.5, rng.random(lps[0].n) < 0.5
    c1, c2 = rng.normal(size=lps[1].n), rng.normal(size=lps[2].n)
    a, kappa = 0.5, 2.0
    c0 = a * kappa * lps[0].c + (1 - a) * np.where(ii, np.where(up, -1.0, 1.0), 0.0)
    with pdhg.Batch(lps, precision=pdhg.FP64, stream=stream.cuda_stream) as b:
        b.solve(tol=1e-300, iter_limit=0, autotune=0)
        for _ in range(first):
            b.set_objective(2, c2)
        with torch.cuda.stream(stream):
            w = torch.rand(4096, 4096, device="cuda")
            for _ in range(20):
                w = w @ w * 1e-3
        b.set_blend(0, up, a, kappa, is_int=ii)
        b.set_objective(1, c1)  # 1.03 MB: all of the buffer
        for q, (r, c) in enumerate(zip(b.solve(tol=1e-300, iter_limit=0, autotune=0), (c0, c1, c2))):
            omega, rel = _expect(lps[q], c)
            assert abs(r["omega"] - omega) <= 1e-9 * omega and abs(r["rel_kkt"] - rel) <= 1e-9 * rel


def test_updates_of_a_captured_stream_are_refused():
    """A caller's graph must not hold launches that read the staging buffer;
    the capture itself goes on, and the handle keeps its objective."""
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    lp = _lp(5100, 3)
    stream = torch.cuda.Stream()
    graph = torch.cuda.CUDAGraph()
    out = torch.zeros(8, device="cuda")
    with pdhg.Batch([lp], precision=pdhg.FP64, stream=stream.cuda_stream) as b:
        b.set_objective(0, lp.c)
        b.solve(tol=1e-300, iter_limit=0, autotune=0)
        torch.cuda.synchronize()
        with torch.cuda.graph(graph, stream=stream):
            out.add_(1.0)
            with pytest.raises(RuntimeError):
                b.set_objective(0, 2.0 * lp.c)
            with pytest.raises(RuntimeError):
                b.set_blend(0, np.ones(lp.n, dtype=bool), 0.5, 1.0)
        for _ in range(3):
            graph.replay()
        torch.cuda.synchronize()
        assert out.tolist() == [3.0] * 8
        r = b.solve(tol=1e-300, iter_limit=0, autotune=0)[0]
        omega, rel = _expect(lp, lp.c)
        assert abs(r["omega"] - omega) <= 1e-9 * omega and abs(r["rel_kkt"] - rel) <= 1e-9 * rel
