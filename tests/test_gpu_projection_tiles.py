"""Tiles of the projections that only certain sizes choose, against the oracle: the gate/up projection on every tile height and
width (odd numbers of column blocks, loads that do not divide evenly over the wavefronts, tiles past the last row and column),
the output projections on 320 x 192 and 256 x 128 tiles, and rows of a power-of-two pitch, whose column tiles start at
different k-tiles and wrap around; float projections on 16 x 16 tiles.  The tiles that the lists name are checked against the planner
without a device (named_tiles).  Tolerance: that of every layer test of the type."""
import pytest

from workloads.configs import ModelShape

from plan_util import F32, SWIGLU, projection_plan
from test_gpu_f32_kernels import test_float_layer as float_layer
from test_gpu_projection_depth import check_layer

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def P():
    import paper_2405_16444_amd as pkg
    return pkg


# (rows, d_ff) over two k-tiles: edges of the tiles in rows and columns; several tiles of every height and width (the lists below name
# the tile of each case and walk more of K)
@pytest.mark.parametrize("n_rows,d_ff", [(1, 7176), (17, 5120), (129, 5120), (65, 28680), (193, 20488), (1, 16392), (100, 16384), (1, 20488),
                                         (128, 20480), (257, 8200), (290, 8192), (129, 24584), (191, 24576), (385, 5128), (500, 5120), (385, 8200),
                                         (512, 8192), (385, 10248), (501, 10240), (257, 16392), (320, 16384), (257, 20488), (319, 20480),
                                         (257, 10248), (384, 10240), (321, 16392), (383, 16384)])
def test_gate_up_tiles(P, n_rows, d_ff):
    check_layer(P, ModelShape(1, 128, 2, 1, 64, d_ff, 1e-5, 1e4, "bf16"), "native", n_rows, 1.0, seed=23 * n_rows + d_ff)


# 8-bit weights
@pytest.mark.parametrize("n_rows,d_ff", [(1, 16400), (128, 16384), (129, 8208), (192, 8192), (129, 16400), (190, 16384), (193, 16400), (256, 16384),
                                         (257, 16400), (320, 16384), (321, 16400), (383, 16384)])
def test_gate_up_tiles_int8(P, n_rows, d_ff):
    check_layer(P, ModelShape(1, 128, 2, 1, 64, d_ff, 1e-5, 1e4, "bf16", weight_format="int8"), "int8", n_rows, 1.0, seed=29 * n_rows + d_ff)


K_WIDTHS = [64, 192, 512]                       # 1, 3 and 8 k-tiles: shorter than the load rings, around their depth, more than twice the deepest of the large tiles
# (tile, rows, d_ff): every tile that a plan can ask for, a last row tile of several but not all rows, a last column tile that is not full
GATE_UP = [((64, 128), 9, 264), ((128, 128), 270, 632), ((128, 160), 9, 16456), ((128, 160), 100, 16392), ((128, 224), 9, 20504), ((192, 128), 270, 5232),
           ((192, 160), 270, 8360), ((192, 224), 580, 13512), ((192, 256), 270, 10936), ((256, 128), 390, 5232), ((256, 160), 580, 5416),
           ((256, 224), 420, 10384), ((256, 256), 390, 10384), ((320, 160), 580, 7256), ((320, 192), 520, 10384), ((384, 128), 270, 10384),
           ((384, 160), 330, 16456)]
GATE_UP_INT8 = [((64, 128), 9, 256), ((128, 128), 150, 5408), ((128, 256), 9, 16448), ((192, 128), 270, 5408), ((192, 160), 150, 16448),
                ((192, 256), 270, 10560), ((256, 160), 200, 16448), ((256, 256), 390, 10560), ((320, 160), 580, 8352), ((384, 160), 330, 16448)]
# (tile, rows, d, d_ff, int8, workgroups that share a tile of the last round), at least 8 k-tiles each: one and several rounds, even
# and odd numbers of column blocks (the last block of an odd one has no partner)
SHARED = [((64, 128), 5, 1536, 528, 0, 3), ((128, 160), 253, 1536, 528, 0, 3), ((384, 160), 330, 1536, 20656, 0, 3), ((64, 128), 5, 1024, 528, 1, 2),
          ((64, 128), 5, 1024, 16512, 1, 2), ((192, 160), 1030, 1536, 528, 1, 3), ((256, 256), 700, 1024, 10592, 1, 2)]
# (tile, rows, d, d_ff, K splits) of the down projection
DOWN = [((320, 192), 520, 6208, 3072, 3), ((128, 256), 270, 8256, 1536, 2), ((256, 128), 390, 5184, 1536, 2)]


def gate_up_model(d, d_ff, int8=0):
    return ModelShape(1, d, 2, 1, 64, d_ff, 1e-5, 1e4, "bf16", weight_format="int8" if int8 else "native")


def named_tiles():
    out = []
    for int8, cases in ((0, GATE_UP), (1, GATE_UP_INT8)):
        out += [(((rows, d, d_ff, int8), {"tile": tile, "shared": 1}), projection_plan(SWIGLU, rows, d_ff, d, w8=int8))
                for tile, rows, d_ff in cases for d in K_WIDTHS]
    out += [(((rows, d, d_ff, int8), {"tile": tile, "shared": shared}), projection_plan(SWIGLU, rows, d_ff, d, w8=int8))
            for tile, rows, d, d_ff, int8, shared in SHARED]
    out += [(((rows, d, d_ff), {"tile": tile, "splits": splits}), projection_plan(F32, rows, d, d_ff)) for tile, rows, d, d_ff, splits in DOWN]
    out += [(((n_rows, 5376, 7168), {"tile": (320, 192), "splits": splits}), projection_plan(F32, n_rows, 5376, 7168)) for n_rows, splits in ((300, 8), (577, 4))]
    return out


@pytest.mark.parametrize("d", K_WIDTHS)
@pytest.mark.parametrize("tile,n_rows,d_ff", GATE_UP)
def test_gate_up_tiles_over_several_k_tiles(P, tile, n_rows, d_ff, d):
    check_layer(P, gate_up_model(d, d_ff), "native", n_rows, 1.0, seed=41 * n_rows + d, std=d ** -0.5)


@pytest.mark.parametrize("d", K_WIDTHS)
@pytest.mark.parametrize("tile,n_rows,d_ff", GATE_UP_INT8)
def test_gate_up_tiles_int8_over_several_k_tiles(P, tile, n_rows, d_ff, d):
    check_layer(P, gate_up_model(d, d_ff, 1), "int8", n_rows, 1.0, seed=43 * n_rows + d, std=d ** -0.5)


@pytest.mark.parametrize("tile,n_rows,d,d_ff,int8,shared", SHARED)
def test_shared_last_round(P, tile, n_rows, d, d_ff, int8, shared):
    check_layer(P, gate_up_model(d, d_ff, int8), "int8" if int8 else "native", n_rows, 1.0, seed=47 * n_rows + d, std=d ** -0.5)


@pytest.mark.parametrize("tile,n_rows,d,d_ff,splits", DOWN)
def test_down_tiles(P, tile, n_rows, d, d_ff, splits):
    check_layer(P, ModelShape(1, d, 2, 1, 64, d_ff, 1e-5, 1e4, "bf16"), "native", n_rows, 1.0, seed=53 * n_rows, std=d ** -0.5)


# down projection, 7168 -> 5376: 320 x 192 tiles in 8 and 4 splits
@pytest.mark.parametrize("n_rows", [300, 577])
def test_output_tiles(P, n_rows):
    check_layer(P, ModelShape(1, 5376, 2, 1, 64, 7168, 1e-5, 1e4, "bf16"), "native", n_rows, 1.0, seed=31 * n_rows, std=5376 ** -0.5)


# K = 4096 of the Q/K/V and gate/up projections (d = 4096), of the output and down projections (64 heads x 64, d_ff = 4096)
@pytest.mark.parametrize("n_rows", [1, 40, 130])
@pytest.mark.parametrize("d,hq,hkv,d_ff", [(4096, 2, 1, 264), (136, 64, 1, 4096)])
def test_staggered_k_ranges(P, n_rows, d, hq, hkv, d_ff):
    check_layer(P, ModelShape(1, d, hq, hkv, 64, d_ff, 1e-5, 1e4, "bf16"), "native", n_rows, 0.9, seed=37 * n_rows + d, std=4096 ** -0.5)


# float 16 x 16 tiles: K shorter than a wavefront's share of a step, at the end of a batch of steps (768) and past it
@pytest.mark.parametrize("rope", ["adjacent", "half"])
@pytest.mark.parametrize("n_rows,d_ff", [(1, 8), (16, 40), (17, 760), (32, 768), (33, 776), (49, 1544)])
def test_small_float_tiles(P, n_rows, d_ff, rope):
    float_layer(P, (136, 3, 1, 64, d_ff, rope, n_rows, 0.7 if n_rows > 20 else 1.0))
