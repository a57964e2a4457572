"""Plans of the projection launches (tile, K split, parked sums), asked of the library's planner without a device."""
import ctypes
import os
import time

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LIB = os.path.join(ROOT, "paper_2405_16444_amd", "libcacheblend.so")
SEG, SWIGLU, F32 = 0, 1, 2


@pytest.fixture(scope="module")
def plan():
    if not os.path.exists(LIB):
        from paper_2405_16444_amd import build
        build.build()
    import torch  # noqa: F401  (the library uses the HIP runtime that torch brings)
    fn = ctypes.CDLL(LIB).cb_internal_projection_plan
    fn.argtypes = [ctypes.c_int] * 8 + [ctypes.c_size_t, ctypes.POINTER(ctypes.c_int)]
    fn.restype = ctypes.c_size_t

    def query(epi, rows, n, k, hl=0, raw=0, w8=0, scratch=2 ** 64 - 1):
        out = (ctypes.c_int * 8)()
        parked = fn(1, epi, rows, n, k, hl, raw, w8, scratch, out)
        return dict(zip(("kind", "bm", "bn", "splits", "tail_splits", "mode", "stagger", "finish"), out), parked=parked)
    return query


@pytest.mark.parametrize("w8", [0, 1])
@pytest.mark.parametrize("epi,n,k,hl", [(SEG, 6144, 4096, 2048), (SWIGLU, 14336, 4096, 0), (F32, 4096, 14336, 0)])
def test_planning_takes_the_same_time_at_any_row_count(plan, epi, n, k, hl, w8):
    """A context's workspace size asks for the plan of every row count up to its maximum (2^24 at most), so the time of one plan must not
    grow with the rows: 20 times is far above what the closed form shows (1) and far below a walk over the row tiles (hundreds)."""
    def seconds(rows):
        best = 1e9
        for _ in range(5):
            t = time.perf_counter()
            for _ in range(50):
                plan(epi, rows, n, k, hl, w8=w8)
            best = min(best, time.perf_counter() - t)
        return best
    assert seconds(1 << 24) < 20 * seconds(100)
