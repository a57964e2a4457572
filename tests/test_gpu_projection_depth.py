"""Projections whose K range is shorter than, as long as and a little longer than the load pipeline is deep (1 .. 8 k-tiles of
64 against 2 .. 6 stages), at the row counts where the tile height changes, bf16 and 8-bit weights.  Tolerance: that of
every bf16 layer test (one rounding of a stored value is 2^-9; a layer's results are a few such roundings deep)."""
import numpy as np
import pytest

from oracle import cacheblend_oracle as O
from workloads import synth
from workloads.configs import ModelShape

from gpu_util import TOL, announce, max_abs_rel, to_np
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
    d = 64 * k_tiles
    model = ModelShape(1, d, k_tiles, 1, 64, 64 * (9 - k_tiles), 1e-5, 1e4, "bf16", weight_format=weights)
    n_suffix = min(3, n_rows)
    n_cand = n_rows - n_suffix
    k = int(n_cand * 0.9)
    announce("projection depth", weights, k_tiles, n_rows, k)
    lw, h, pos, kc, vc = layer_case(model, n_rows + 40, n_rows, n_suffix, seed=13 * n_rows + k_tiles)
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
