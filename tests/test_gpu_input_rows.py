"""The launch that takes a call's input rows in (float copy, positions, first RMSNorm) at the widths where its register layout
changes, and layers without a check, which keep the positions where they are, before and after a checked one.  The layer-by-layer
calls normalise and number the rows themselves, so equality with them is exact; against the oracle the usual tolerance, with weights of standard
deviation d^-1/2: with the small models' 0.07 queries and keys are of order 0.07 sqrt(d) = 3.2 .. 6.3, scores of order 80 .. 300, and a
bf16 rounding of a query (2^-9) moves a score by 0.2 .. 0.6, a probability by as much."""
import numpy as np
import pytest
import torch

from oracle import cacheblend_oracle as O
from workloads.configs import ModelShape

from gpu_util import TOL, announce, cache_tensors, dev_layers, max_abs_rel, to_np
from test_gpu_parity import e2e_case, run_prefill

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def P():
    import paper_2405_16444_amd as pkg
    return pkg


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("d", [8, 2048, 2056, 4096, 4104, 8192, 8200])
def test_input_rows_and_unchecked_layers(P, d, dtype):
    model = ModelShape(3, d, 2, 1, 64, 64, 1e-5, 1e4, dtype)
    announce("input rows", d, dtype)
    w, layers, x, npl, xn, kpre, vpre = e2e_case(model, (12, 9), 3, seed=400 + d, std=max(d, 200) ** -0.5)
    keep = [21, 21, 8]                                   # layers 0 and 1 keep every row
    out, kg, vg = run_prefill(P, w, layers, x, kpre, vpre, keep)
    ctx = P.cb_create(model, w.n_tokens)
    k2, v2 = cache_tensors(w, kpre, vpre)
    dl = dev_layers(layers)
    P.cb_realign_rope(ctx, k2, 0, 3, [0, 12, 21])
    h, pos = x.cuda().float(), torch.arange(w.n_tokens, dtype=torch.int32, device="cuda")
    for l in range(3):
        h, pos, _ = P.cb_fuse_layer(ctx, l, dl[l], h, pos, w.n_suffix, k2[l], v2[l], keep[l])
        assert torch.equal(pos[:keep[l]], out.sel[l])
    torch.cuda.synchronize()
    P.cb_destroy(ctx)
    assert torch.equal(h[-w.n_suffix:], out.final_hidden)
    for l in range(3):
        assert torch.equal(k2[l], kg[l]) and torch.equal(v2[l], vg[l])
    sel = [s.cpu().numpy().astype(np.int64) for s in out.sel]
    ref = O.fuse_prefill(xn, npl, model, w.chunk_lens, w.n_suffix, kpre, vpre, keep, forced_sel=sel, kv_round=O.storage_round(dtype))
    assert max_abs_rel(to_np(out.final_hidden), ref.final_hidden) < TOL[dtype]
    for l in range(3):
        assert max_abs_rel(to_np(kg[l]), ref.K[l]) < TOL[dtype] and max_abs_rel(to_np(vg[l]), ref.V[l]) < TOL[dtype]
