"""The library's host runtime without a GPU: tests/host/runtime_driver.cpp
replaces the HIP runtime by one that queues work until something waits for it
and checks what the library launches (sizes, buffers, staged data)."""
import os
import subprocess
import tempfile

import pytest

from paper_2307_03466_amd import pdhg

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def driver():
    if not os.path.exists(pdhg.LIB_PATH):
        import __graft_entry__
        __graft_entry__.build()
    exe = os.path.join(tempfile.mkdtemp(), "runtime_driver")
    subprocess.check_call(["g++", "-O1", "-std=c++17", "-w", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
                           "-o", exe, os.path.join(ROOT, "tests", "host", "runtime_driver.cpp"), "-rdynamic",
                           pdhg.LIB_PATH, "-Wl,--allow-shlib-undefined",
                           "-Wl,-rpath," + os.path.dirname(pdhg.LIB_PATH), "-lpthread"])

    def run(*args):
        r = subprocess.run([exe, *map(str, args)], capture_output=True, text=True, timeout=110)
        assert r.returncode == 0 and r.stdout.strip() == "ok", r.stdout[-2000:] + r.stderr[-2000:]
    return run


@pytest.mark.parametrize("n,objectives", [(120000, 0), (131072, 0), (40000, 1), (16384, 1), (17, 1)])
def test_updates_read_their_own_staged_bits(driver, n, objectives):
    """Rounding and integer bits of one update are staged together: the
    buffer starting over between the two would hand the first to later
    updates while the stream is behind."""
    driver("blends", n, 400, objectives)


@pytest.mark.parametrize("small,rows,cols", [(16384, 1000000, 1100000), (65536, 300000, 530000), (3, 2, 5)])
def test_one_large_lp_among_many_small_ones(driver, small, rows, cols):
    """No launch beyond 2^32 threads, no buffer of instances x the largest."""
    driver("uneven", small, rows, cols)


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("call", ["layout:0,4,0,4", "layout:0,8,0,-16", "layout:2,8,4,8", "layout:-1,8,-1,8",
                                  "layout:-2,4,-2,4", "layout:-3,8,-3,8", "layout:-6,8,-7,4", "solve"])
def test_failed_allocations(driver, call, precision):
    """Any allocation of a layout change or of a solve fails: the same call
    made again works, and so does a solve without it."""
    driver("allocations", call, precision)


@pytest.mark.parametrize("period", [1, 3, 1024])
def test_largest_iteration_limit(driver, period):
    """The number of checks of a fused solve does not overflow: something is
    launched, and the solve ends."""
    driver("limit", period)


@pytest.mark.parametrize("n", [50, 131000, 140000])
def test_updates_of_a_captured_stream_are_refused(driver, n):
    """Staged in place, staged whole, and larger than the staging buffer."""
    driver("captured", n)


def test_the_graph_is_not_the_loops_time(driver):
    driver("slow_graph")
