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


@pytest.mark.parametrize("value", [float("nan"), float("inf")], ids=str)
@pytest.mark.parametrize("dh,n_rows,n_tokens", [(64, 40, 90), (64, 300, 700), (128, 33, 70)])
def test_a_bad_value_row_reaches_only_the_rows_that_see_it(P, dh, n_rows, n_tokens, value):
    """A reused value row that is not finite belongs to the queries at and after its position; the queries before it that
    share an attention block with some of those match the oracle on a clean cache, which never shows them that row."""
    model = ModelShape(1, 256, 4, 2, dh, 688, 1e-5, 1e4, "f32")
    lw, h, pos, kc, vc = layer_case(model, n_tokens, n_rows, 2, seed=dh + n_rows, std=0.05)
    h_ref, _, _, _, _ = oracle_layer(model, lw, h, pos, kc, vc, 2, n_rows - 2, None)
    reused = np.setdiff1d(np.arange(n_tokens), pos.numpy())
    for at in (reused[0], reused[len(reused) // 3], reused[len(reused) // 2], reused[-1]):
        announce("float attention, bad value row", dh, n_rows, int(at), value)
        bad = vc.clone()
        bad[int(at), :, dh - 1] = value
        h_out, pos_out, _, _, _ = run_layer_both(P, model, lw, h, pos, kc, bad, 2, n_rows - 2, want_dev=False)
        before = pos_out.numpy() < at
        assert max_abs_rel(to_np(h_out)[before], h_ref[before]) < TOL["f32"]
        assert not np.isfinite(h_out.numpy()[~before]).all(axis=1).any()
