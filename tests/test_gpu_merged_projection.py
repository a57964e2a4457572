"""K, V and Q of a layer in one projection launch (or, where that is estimated to be slower, in two): key/value columns
(operand pairs) that fill one column tile of 128 and several, row counts around the tile edges of both kinds of columns, with
a selection (Q is then computed for every candidate and read through the kept list) and without one, both rotary orders and
8-bit weights.  Column tiles of 256 meet in test_gpu_projection_depth.py and, with a selection, in the real-width tests."""
import numpy as np
import pytest

from oracle import cacheblend_oracle as O
from workloads import synth
from workloads.configs import ModelShape

from gpu_util import TOL, announce, max_abs_rel, to_np
from test_gpu_parity import layer_case, oracle_layer, run_layer_both

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def P():
    import paper_2405_16444_amd as pkg
    return pkg


@pytest.mark.parametrize("d,hq,hkv,dh,rope", [(256, 4, 1, 64, "adjacent"),       # 128 pair columns: half of the wide tile
                                              (512, 8, 2, 64, "half"),            # 256: one wide tile
                                              (512, 6, 3, 128, "half"),           # 768: three
                                              (320, 5, 5, 64, "adjacent")])       # 640: no whole number of wide tiles
@pytest.mark.parametrize("n_rows,k_share", [(1, 1.0), (17, 0.5), (64, 0.95), (65, 0.95), (129, 1.0), (257, 0.9), (515, 0.97)])
def test_layer_matches_the_oracle(P, d, hq, hkv, dh, rope, n_rows, k_share):
    model = ModelShape(1, d, hq, hkv, dh, 704, 1e-5, 1e4, "bf16", rope_layout=rope)
    n_suffix = min(3, n_rows)
    n_cand = n_rows - n_suffix
    k = int(n_cand * k_share)
    announce("merged projection", d, hq, hkv, dh, rope, n_rows, k)
    lw, h, pos, kc, vc = layer_case(model, n_rows + 40, n_rows, n_suffix, seed=31 * n_rows + d)
    check = k < n_cand
    h_out, pos_out, dev, kg, vg = run_layer_both(P, model, lw, h, pos, kc, vc, n_suffix, k, want_dev=check)
    forced = pos.numpy()[:n_cand][O.top_k_indices(dev.numpy(), k)] if check else None
    h_ref, pos_ref, dev_ref, ko, vo = oracle_layer(model, lw, h, pos, kc, vc, n_suffix, k, forced)
    tol = TOL["bf16"]
    assert np.array_equal(pos_out.numpy(), pos_ref)
    if check:
        assert max_abs_rel(dev.numpy(), dev_ref) < tol
    assert max_abs_rel(to_np(kg), ko) < tol and max_abs_rel(to_np(vg), vo) < tol
    assert max_abs_rel(to_np(h_out), h_ref) < tol


@pytest.mark.parametrize("n_rows,k_share", [(33, 0.9), (300, 1.0)])
def test_int8_weights(P, n_rows, k_share):
    model = ModelShape(1, 512, 8, 2, 64, 704, 1e-5, 1e4, "bf16", weight_format="int8")
    lw, h, pos, kc, vc = layer_case(model, n_rows + 40, n_rows, 3, seed=77 + n_rows)
    q = synth.quantize_int8(lw)
    k = int((n_rows - 3) * k_share)
    announce("merged projection, 8-bit weights", n_rows, k)
    check = k < n_rows - 3
    h_out, pos_out, dev, kg, vg = run_layer_both(P, model, q, h, pos, kc, vc, 3, k, want_dev=check)
    forced = pos.numpy()[:n_rows - 3][O.top_k_indices(dev.numpy(), k)] if check else None
    deq = O.dequantize_int8({name: synth.to_f64(t) for name, t in q.items()})
    ko, vo = to_np(kc), to_np(vc)
    h_ref, pos_ref, _, _ = O.fuse_layer(deq, model, to_np(h), pos.numpy(), 3, ko, vo, k, forced_sel=forced,
                                        kv_round=O.storage_round("bf16"))
    assert np.array_equal(pos_out.numpy(), pos_ref)
    assert max_abs_rel(to_np(kg), ko) < TOL["bf16"] and max_abs_rel(to_np(vg), vo) < TOL["bf16"]
    assert max_abs_rel(to_np(h_out), h_ref) < TOL["bf16"]


# The room for K, V and Q in one launch does not hang on what other projections of the row count park (their plans changed, and with them a layer
# of 32 key/value heads at 1320 rows fell back to two launches: 263 -> 287 us)
@pytest.mark.parametrize("n_rows,d,hq,hkv,dh,d_ff", [(1320, 2048, 32, 32, 64, 5632), (700, 1024, 16, 16, 64, 2816)])
def test_q_rides_along(P, n_rows, d, hq, hkv, dh, d_ff):
    import torch
    model = ModelShape(1, d, hq, hkv, dh, d_ff, 1e-5, 1e4, "bf16")
    announce("merged projection, launches", n_rows, d, hq, hkv)
    lw, h, pos, kc, vc = layer_case(model, n_rows + 40, n_rows, 16, seed=n_rows, std=d ** -0.5)
    ctx = P.cb_create(model, n_rows + 40)
    P.cb_profile_enable(ctx, 1)
    P.cb_fuse_layer(ctx, 0, {k: v.cuda() for k, v in lw.items()}, h.cuda(), pos.cuda(), 16, kc.cuda(), vc.cuda(), int((n_rows - 16) * 0.9))
    torch.cuda.synchronize()
    assert P.cb_profile_read(ctx)["gemm"]["launches"] == 4
    P.cb_destroy(ctx)
