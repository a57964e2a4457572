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


def measured():
    for line in open(os.path.join(ROOT, "profiles", "projection_tiles.tsv")):
        if not line.startswith("#"):
            kind, *numbers, pairs = line.rstrip("\n").split("\t")
            yield kind, *map(int, numbers), {k: float(v) for k, v in (p.split("=") for p in pairs.split())}


# problems of the table, and what the chosen pair may take over the best one: on average, and any one problem (1.2: not among the pairs
# within 20 %).  The averages are what the models show, rounded up to half a percent, and repeats of one pair differ by 3 % alone; single problems are
# a matter of 1 .. 3 us in launches of 10 .. 25.
CHOICES = {
    "K and V alone": (lambda kind, n, hl, w8: kind == "seg" and n == hl, 1.015, 1.18),
    "output and down": (lambda kind, n, hl, w8: kind == "f32", 1.015, 1.21),
    "K, V and Q": (lambda kind, n, hl, w8: kind == "seg" and 0 < hl < n, 1.01, 1.15),
    "gate and up": (lambda kind, n, hl, w8: kind == "gate_up" and not w8, 1.01, 1.11),
    "gate and up, int8": (lambda kind, n, hl, w8: kind == "gate_up" and w8, 1.01, 1.18),
    "Q alone": (lambda kind, n, hl, w8: kind == "seg" and hl == 0, 1.02, 1.12),
}


@pytest.mark.parametrize("which", CHOICES)
def test_chosen_pairs_against_measured_times(plan, which):
    wanted, mean, most = CHOICES[which]
    ratios = []
    for kind, n, k, hl, checked, w8, rows, pairs in measured():
        if not wanted(kind, n, hl, w8):
            continue
        p = plan({"seg": SEG, "f32": F32, "gate_up": SWIGLU}[kind], rows, n, k, hl, checked, w8)
        chosen = f"{p['bm']}x{p['bn']}/{p['tail_splits'] if kind == 'gate_up' else p['splits']}"
        ratios.append((pairs.get(chosen, 1.2 * min(pairs.values())) / min(pairs.values()), n, k, rows, chosen))
    assert len(ratios) > 100
    product = 1.0
    for r in ratios:
        product *= r[0]
    assert product ** (1 / len(ratios)) < mean and max(ratios)[0] < most, sorted(ratios)[-5:]
