"""Tiles of the projections that only certain sizes choose, against the oracle: the gate/up projection on every tile height and
width (odd numbers of column blocks, loads that do not divide evenly over the wavefronts, tiles past the last row and column),
the output projections on 192 x 224 and 320 x 192 tiles, and rows of a power-of-two pitch, whose column tiles start at
different k-tiles and wrap around; float projections on 16 x 16 tiles.  Tolerance: that of every layer test of the type."""
import pytest

from workloads.configs import ModelShape

from test_gpu_f32_kernels import test_float_layer as float_layer
from test_gpu_projection_depth import check_layer

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def P():
    import paper_2405_16444_amd as pkg
    return pkg


# (rows, d_ff): the smallest problem that takes the tile, and one a few rows or 8 columns off.
# bf16: 64, 128, 192 x 128; 192 x 256, 256 x 256; 128 x 160, 128 x 224; 192 x 160, 192 x 224; 256 x 128, 160, 224;
# 320 x 160, 320 x 192; 384 x 128, 384 x 160
@pytest.mark.parametrize("n_rows,d_ff", [(1, 7176), (17, 5120), (129, 5120), (65, 28680), (193, 20488), (1, 16392), (100, 16384), (1, 20488),
                                         (128, 20480), (257, 8200), (290, 8192), (129, 24584), (191, 24576), (385, 5128), (500, 5120), (385, 8200),
                                         (512, 8192), (385, 10248), (501, 10240), (257, 16392), (320, 16384), (257, 20488), (319, 20480),
                                         (257, 10248), (384, 10240), (321, 16392), (383, 16384)])
def test_gate_up_tiles(P, n_rows, d_ff):
    check_layer(P, ModelShape(1, 128, 2, 1, 64, d_ff, 1e-5, 1e4, "bf16"), "native", n_rows, 1.0, seed=23 * n_rows + d_ff)


# 8-bit weights: 128 x 256; 192 x 128, 160; 256 x 160; 320 x 160; 384 x 160
@pytest.mark.parametrize("n_rows,d_ff", [(1, 16400), (128, 16384), (129, 8208), (192, 8192), (129, 16400), (190, 16384), (193, 16400), (256, 16384),
                                         (257, 16400), (320, 16384), (321, 16400), (383, 16384)])
def test_gate_up_tiles_int8(P, n_rows, d_ff):
    check_layer(P, ModelShape(1, 128, 2, 1, 64, d_ff, 1e-5, 1e4, "bf16", weight_format="int8"), "int8", n_rows, 1.0, seed=29 * n_rows + d_ff)


# down projection, 7168 -> 5376: 192 x 224 tiles in 5 splits, 320 x 192 tiles in 4
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
