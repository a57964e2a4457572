"""Plans of the projection launches (tile, K split, parked sums), asked of the library's planner without a device."""
import os
import time

import pytest

from plan_util import F32, ROOT, SEG, SWIGLU, projection_plan


@pytest.mark.parametrize("w8", [0, 1])
@pytest.mark.parametrize("epi,n,k,hl", [(SEG, 6144, 4096, 2048), (SWIGLU, 14336, 4096, 0), (F32, 4096, 14336, 0)])
def test_planning_takes_the_same_time_at_any_row_count(epi, n, k, hl, w8):
    """A context's workspace size asks for the plan of every row count up to its maximum (2^24 at most), so the time of one plan must not
    grow with the rows: 20 times is far above what the closed form shows (1) and far below a walk over the row tiles (hundreds)."""
    def seconds(rows):
        best = 1e9
        for _ in range(5):
            t = time.perf_counter()
            for _ in range(50):
                projection_plan(epi, rows, n, k, hl, w8=w8)
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
def test_chosen_pairs_against_measured_times(which):
    wanted, mean, most = CHOICES[which]
    ratios = []
    for kind, n, k, hl, checked, w8, rows, pairs in measured():
        if not wanted(kind, n, hl, w8):
            continue
        p = projection_plan({"seg": SEG, "f32": F32, "gate_up": SWIGLU}[kind], rows, n, k, hl, checked, w8)
        chosen = f"{p['bm']}x{p['bn']}/{p['shared'] if kind == 'gate_up' else p['splits']}"
        ratios.append((pairs.get(chosen, 1.2 * min(pairs.values())) / min(pairs.values()), n, k, rows, chosen))
    assert len(ratios) > 100
    product = 1.0
    for r in ratios:
        product *= r[0]
    assert product ** (1 / len(ratios)) < mean and max(ratios)[0] < most, sorted(ratios)[-5:]


# one round of few workgroups, each with a long K: alone they took up to three times as long (1024 x 8192 at 16 rows 59 us, shared by four 21)
@pytest.mark.parametrize("w8", [0, 1])
@pytest.mark.parametrize("rows,n,k", [(1, 512, 8192), (64, 512, 8192), (16, 272, 4096), (128, 8192, 3072)])
def test_a_single_part_filled_round_is_shared(rows, n, k, w8):
    assert projection_plan(SWIGLU, rows, n, k, w8=w8)["shared"] > 1


def test_gpu_cases_take_the_tiles_they_name():
    import test_gpu_projection_depth as depth
    import test_gpu_projection_tiles as tiles
    wrong = []
    for case, got in tiles.named_tiles() + depth.named_tiles():
        if any(got[key] != value for key, value in case[1].items()):
            wrong.append((case, {key: got[key] for key in case[1]}))
    assert not wrong, wrong


def test_every_tile_of_the_gate_up_projection_has_a_case_of_several_k_tiles():
    """What plans can ask for, found by asking over rows and columns, against the GPU cases: 3, 5 and 8 k-tiles of each tile."""
    import test_gpu_projection_tiles as tiles
    for w8, cases in ((0, tiles.GATE_UP), (1, tiles.GATE_UP_INT8)):
        asked = {projection_plan(SWIGLU, rows, n, 4096, w8=w8)["tile"]
                 for rows in (1, 40, 100, 150, 200, 270, 330, 390, 420, 520, 580, 700, 1100, 2000) for n in range(512, 30000, 272)}
        assert asked <= {case[0] for case in cases}, asked - {case[0] for case in cases}


# (rows, columns, K, most MB of parked sums).  Workspaces are sized for the parked sums; 184, 184 and 551 MB bought nothing over these
@pytest.mark.parametrize("rows,n,k,most", [(1600, 7168, 20480, 140), (2048, 7168, 20480, 120), (4200, 8192, 28672, 420)])
def test_large_launches_park_what_pays(rows, n, k, most):
    assert projection_plan(F32, rows, n, k)["parked"] * 4e-6 <= most
