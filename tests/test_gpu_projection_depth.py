"""Projections whose K range is shorter than, as long as and a little longer than the load pipeline is deep, bf16 and 8-bit
weights: the 128-column tiles (1 .. 8 k-tiles of 64 against 3 .. 6 stages) at the row counts where the tile height changes,
and the 256-column tiles (2 activation and 3 weight stages or 3 .. 5 of both) at row and column counts that fill the chip
with them.  Tolerance: that of every bf16 layer test (one rounding of a stored value is 2^-9; a layer's results are a few
such roundings deep)."""
import numpy as np
import pytest

from oracle import cacheblend_oracle as O
from workloads import synth
from workloads.configs import ModelShape

from gpu_util import TOL, announce, max_abs_rel, to_np
from plan_util import F32, SEG, SWIGLU, projection_plan
from test_gpu_parity import layer_case, run_layer_both

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def P():
    import paper_2405_16444_amd as pkg
    return pkg


@pytest.mark.parametrize("weights", ["native", "int8"])
@pytest.mark.parametrize("k_tiles", [1, 2, 3, 4, 5, 6, 7, 8])
@pytest.mark.parametrize("n_rows", [1, 33, 64, 65, 129, 193, 257])
def test_layer_matches_the_oracle(P, weights, k_tiles, n_rows):
    check_layer(P, ModelShape(1, 64 * k_tiles, k_tiles, 1, 64, 64 * (9 - k_tiles), 1e-5, 1e4, "bf16", weight_format=weights),
                weights, n_rows, 0.9, seed=13 * n_rows + k_tiles)


def check_layer(P, model, weights, n_rows, k_share, seed, std=0.07):
    n_suffix = min(3, n_rows)
    n_cand = n_rows - n_suffix
    k = int(n_cand * k_share)
    announce("projection depth", model, n_rows, k)
    lw, h, pos, kc, vc = layer_case(model, n_rows + 40, n_rows, n_suffix, seed=seed, std=std)
    q = synth.quantize_int8(lw) if weights == "int8" else lw
    check = k < n_cand
    h_out, pos_out, dev, kg, vg = run_layer_both(P, model, q, h, pos, kc, vc, n_suffix, k, want_dev=check)
    forced = pos.numpy()[:n_cand][O.top_k_indices(dev.numpy(), k)] if check else None
    ref = {name: synth.to_f64(t) for name, t in q.items()}
    if weights == "int8":
        ref = O.dequantize_int8(ref)
    ko, vo = to_np(kc), to_np(vc)
    h_ref, pos_ref, _, _ = O.fuse_layer(ref, model, to_np(h), pos.numpy(), n_suffix, ko, vo, k, forced_sel=forced,
                                        kv_round=O.storage_round("bf16"))
    assert np.array_equal(pos_out.numpy(), pos_ref)
    assert max_abs_rel(to_np(kg), ko) < TOL["bf16"] and max_abs_rel(to_np(vg), vo) < TOL["bf16"]
    assert max_abs_rel(to_np(h_out), h_ref) < TOL["bf16"]


# Q/K/V and gate/up over 1 .. 4 k-tiles.  Tiles: 513 rows 192 x 160 gate/up; 1024 rows 256 x 256 gate/up, and for Q/K/V 256 x 256
# with 2560 columns of operand pairs (ten wide tiles) or 128 x 256 with 256 of them (one); 1280 rows 192 x 256 Q/K/V (where Q rides along).
@pytest.mark.parametrize("weights,k_tiles", [("native", 1), ("native", 2), ("native", 3), ("native", 4), ("int8", 2), ("int8", 4)])
@pytest.mark.parametrize("n_rows,hq,hkv,dh", [(513, 20, 10, 128), (1024, 20, 10, 128), (1024, 64, 2, 64), (1280, 32, 2, 128)])
def test_wide_tiles_match_the_oracle(P, weights, k_tiles, n_rows, hq, hkv, dh):
    model = ModelShape(1, 64 * k_tiles, hq, hkv, dh, 6400, 1e-5, 1e4, "bf16", weight_format=weights,
                       rope_layout="half" if k_tiles % 2 else "adjacent")
    check_layer(P, model, weights, n_rows, 1.0, seed=17 * n_rows + k_tiles)


# The output projection (K = heads x 64) on 256 x 128 tiles at 1024 rows and on 192 x 256 tiles at 1500, the down projection
# (K = 64) on the same.  Weights of standard deviation 6144^-1/2: with the small models' 0.07, queries and keys are of order 5.5
# and scores of order 240, and rounding the oracle's own queries to bf16 moves its result by 0.052 (by 9e-5 with these).
@pytest.mark.parametrize("k_tiles", [1, 2, 3, 4])
@pytest.mark.parametrize("n_rows", [1024, 1500])
def test_wide_output_tiles_match_the_oracle(P, k_tiles, n_rows):
    check_layer(P, ModelShape(1, 6144, k_tiles, 1, 64, 64, 1e-5, 1e4, "bf16"), "native", n_rows, 1.0, seed=19 * n_rows + k_tiles,
                std=6144 ** -0.5)


# (tile, rows, d, weights) of the output (K = heads x 64) and the down projection (K = 64) over few k-tiles
OUTPUT = [((256, 128), 580, 8256, "native"), ((192, 256), 1030, 6208, "native"), ((256, 256), 1290, 8256, "native"), ((192, 128), 1290, 2112, "native"),
          ((128, 256), 1290, 2112, "int8"), ((192, 256), 1290, 4160, "int8"), ((256, 256), 1290, 8256, "int8")]


def named_tiles():
    out = []
    for k in (64, 128, 192, 256):
        out += [((("gate_up", rows, k), {"tile": tile}), projection_plan(SWIGLU, rows, 6400, k)) for rows, tile in ((513, (192, 160)), (1024, (256, 256)))]
        out += [((("q/k/v", rows, n, k), {"tile": tile}), projection_plan(SEG, rows, n, k, hl))
                for rows, n, hl, tile in ((1024, 5120, 2560, (256, 256)), (1024, 4352, 256, (128, 256)), (1280, 4608, 512, (192, 256)))]
        out += [((("output", rows, k), {"tile": tile}), projection_plan(F32, rows, 6144, k)) for rows, tile in ((1024, (256, 128)), (1500, (192, 256)))]
        out += [((("output", rows, d, weights, k), {"tile": tile}), projection_plan(F32, rows, d, k, w8=int(weights == "int8")))
                for tile, rows, d, weights in OUTPUT]
    return out


@pytest.mark.parametrize("k_tiles", [1, 3, 4])
@pytest.mark.parametrize("tile,n_rows,d,weights", OUTPUT)
def test_output_tiles_of_few_k_tiles(P, tile, n_rows, d, weights, k_tiles):
    check_layer(P, ModelShape(1, d, k_tiles, 1, 64, 64, 1e-5, 1e4, "bf16", weight_format=weights), weights, n_rows, 1.0, seed=23 * n_rows + k_tiles,
                std=d ** -0.5)
