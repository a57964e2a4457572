"""Float models: row counts around the edges of the 16-query attention blocks and of the 32- and 64-row projection
tiles, inner widths that are no multiple of the 64-deep stage, both head sizes and rotary orders, key counts that leave
some of a workgroup's wavefronts without a tile.  Tolerance: the float bound of every parity test."""
import numpy as np
import pytest

from oracle import cacheblend_oracle as O
from workloads.configs import ModelShape

from gpu_util import TOL, announce, max_abs_rel, to_np
from test_gpu_parity import layer_case, oracle_layer, run_layer_both

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def P():
    import paper_2405_16444_amd as pkg
    return pkg


CASES = [(256, 4, 2, 64, 688, rope, n, k) for rope in ("adjacent", "half")
         for n, k in [(1, 1.0), (15, 1.0), (17, 0.5), (33, 0.9), (65, 0.2), (300, 0.95)]]
CASES += [(328, 6, 2, 128, 1000, rope, n, k) for rope in ("adjacent", "half") for n, k in [(31, 1.0), (64, 0.9), (130, 0.3)]]
CASES += [(512, 8, 4, 64, 1408, "adjacent", 2100, 0.98)]        # enough rows for the 64 x 64 tiles


@pytest.mark.parametrize("case", CASES, ids=lambda c: f"d{c[0]}_h{c[1]}/{c[2]}x{c[3]}_f{c[4]}_{c[5]}_r{c[6]}_k{c[7]}")
def test_float_layer(P, case):
    d, hq, hkv, dh, f, rope, n_rows, k_share = case
    model = ModelShape(1, d, hq, hkv, dh, f, 1e-5, 1e4, "f32", rope_layout=rope)
    n_suffix = min(2, n_rows)
    n_cand = n_rows - n_suffix
    k = int(n_cand * k_share)
    announce("float layer", case)
    lw, h, pos, kc, vc = layer_case(model, n_rows + 25, n_rows, n_suffix, seed=13 * n_rows + d, std=0.05)
    check = k < n_cand
    h_out, pos_out, dev, kg, vg = run_layer_both(P, model, lw, h, pos, kc, vc, n_suffix, k, want_dev=check)
    forced = pos.numpy()[:n_cand][O.top_k_indices(dev.numpy(), k)] if check else None
    h_ref, pos_ref, dev_ref, ko, vo = oracle_layer(model, lw, h, pos, kc, vc, n_suffix, k, forced)
    tol = TOL["f32"]
    assert np.array_equal(pos_out.numpy(), pos_ref)
    if check:
        assert max_abs_rel(dev.numpy(), dev_ref) < tol
    assert max_abs_rel(to_np(kg), ko) < tol and max_abs_rel(to_np(vg), vo) < tol
    assert max_abs_rel(to_np(h_out), h_ref) < tol
