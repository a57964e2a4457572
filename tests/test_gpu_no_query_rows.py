"""Calls without query rows, where nothing reads the last layer's output and only its keys and values are computed:
the producer (several ragged chunks, more cache rows than tokens, inputs in the storage type and in float) and a batched
call whose requests have no suffix."""
from dataclasses import replace

import numpy as np
import pytest
import torch

from oracle import cacheblend_oracle as O
from paper_2405_16444_amd import producer
from workloads import synth

from gpu_util import TOL, announce, dev_layers, max_abs_rel, to_np
from test_gpu_parity import MODELS, e2e_case

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def P():
    import paper_2405_16444_amd as pkg
    return pkg


@pytest.mark.parametrize("name,lens,extra", [("f32", (1, 40, 33), 0), ("bf16", (70, 1, 129), 5), ("bf16_g7", (64,), 300)])
@pytest.mark.parametrize("as_float", [False, True])
def test_producer(P, name, lens, extra, as_float):
    model = replace(MODELS[name], n_layers=3)
    announce("producer", name, lens, extra, as_float)
    w, layers, x, npl, xn, kpre, vpre = e2e_case(model, lens, 2, seed=170 + extra)
    ctx = P.cb_create(model, w.n_tokens)
    xc = x[:w.n_ctx].float() if as_float else x[:w.n_ctx]
    ks, vs = producer.chunk_prefill(ctx, dev_layers(layers), xc.cuda(), lens, w.n_ctx + extra)
    torch.cuda.synchronize()
    P.cb_destroy(ctx)
    for l in range(3):
        for got, ref in ((ks[l], kpre[l]), (vs[l], vpre[l])):
            assert got.shape[0] == w.n_ctx + extra and not got[w.n_ctx:].any()
            assert max_abs_rel(to_np(got[:w.n_ctx].cpu()), ref) < TOL[model.dtype], f"layer {l}"


def test_producer_takes_a_longer_list_of_layers(P):
    """The first n_layers entries are the model's; what follows them is not looked at."""
    model = replace(MODELS["bf16"], n_layers=2)
    announce("producer, longer list of layers")
    w, layers, x, npl, xn, kpre, vpre = e2e_case(model, (30, 41), 2, seed=190)
    ctx = P.cb_create(model, w.n_tokens)
    dl = dev_layers(layers)
    for longer in (dl + [dl[0]], tuple(dl) + (None,)):
        ks, vs = producer.chunk_prefill(ctx, longer, x[:w.n_ctx].cuda(), (30, 41), w.n_ctx)
        torch.cuda.synchronize()
        assert len(ks) == len(vs) == 2
        for l in range(2):
            assert max_abs_rel(to_np(ks[l].cpu()), kpre[l]) < TOL["bf16"]
            assert max_abs_rel(to_np(vs[l].cpu()), vpre[l]) < TOL["bf16"]
    P.cb_destroy(ctx)


def test_producer_takes_16_bit_rows_at_any_address(P):
    model = replace(MODELS["bf16"], n_layers=2)
    announce("producer, input not on a 16-byte boundary")
    w, layers, x, npl, xn, kpre, vpre = e2e_case(model, (30, 41), 2, seed=200)
    ctx = P.cb_create(model, w.n_tokens)
    xc = torch.empty(w.n_ctx * model.d_model + 8, dtype=torch.bfloat16, device="cuda")
    for shift in (1, 4):
        xs = xc[shift:shift + w.n_ctx * model.d_model].view(w.n_ctx, model.d_model)
        xs.copy_(x[:w.n_ctx])
        assert xs.data_ptr() % 16 == 2 * shift
        ks, vs = producer.chunk_prefill(ctx, dev_layers(layers), xs, (30, 41), w.n_ctx)
        torch.cuda.synchronize()
        for l in range(2):
            assert max_abs_rel(to_np(ks[l].cpu()), kpre[l]) < TOL["bf16"]
            assert max_abs_rel(to_np(vs[l].cpu()), vpre[l]) < TOL["bf16"]
    P.cb_destroy(ctx)


@pytest.mark.parametrize("extra", [0, 3])
def test_every_layer_of_the_producer_is_a_tensor_of_its_own(P, extra, tmp_path):
    """Keeping or saving one layer's K keeps or saves that layer's K."""
    model = replace(MODELS["bf16"], n_layers=3)
    announce("producer, storage of the layers", extra)
    w, layers, x, npl, xn, kpre, vpre = e2e_case(model, (30, 41), 2, seed=210)
    ctx = P.cb_create(model, w.n_tokens)
    ks, vs = producer.chunk_prefill(ctx, dev_layers(layers), x[:w.n_ctx].cuda(), (30, 41), w.n_ctx + extra)
    size = (w.n_ctx + extra) * model.kv_dim * 2
    assert all(t.untyped_storage().nbytes() == size and t.storage_offset() == 0 for t in ks + vs)
    torch.save(ks[1], tmp_path / "k1.pt")
    assert (tmp_path / "k1.pt").stat().st_size < size + 4096
    assert torch.equal(torch.load(tmp_path / "k1.pt", weights_only=True), ks[1])
    P.cb_destroy(ctx)


def test_batched_requests_without_a_suffix(P):
    model = replace(MODELS["bf16"], n_layers=3)
    announce("batched, no suffix")
    reqs = [e2e_case(model, lens, 0, seed=180) for lens in ((60, 81), (33, 40, 20))]     # one seed: the same weights
    layers = reqs[0][1]
    stride = max(r[0].n_ctx for r in reqs)
    dt = synth.storage_dtype(model)
    kc = [torch.zeros((2 * stride, model.n_kv_heads, model.head_dim), dtype=dt) for _ in range(3)]
    vc = [torch.zeros_like(t) for t in kc]
    for b, (w, _, _, _, _, kpre, vpre) in enumerate(reqs):
        for l in range(3):
            kc[l][b * stride:b * stride + w.n_ctx] = torch.from_numpy(kpre[l]).to(dt)
            vc[l][b * stride:b * stride + w.n_ctx] = torch.from_numpy(vpre[l]).to(dt)
    kg, vg = [t.cuda() for t in kc], [t.cuda() for t in vc]
    keep = [[r[0].n_ctx, r[0].n_ctx // 2, r[0].n_ctx // 4] for r in reqs]
    ctx = P.cb_create(model, stride)
    out = P.cb_fuse_prefill_batched(ctx, dev_layers(layers), torch.cat([r[2] for r in reqs]).cuda(),
                                    [r[0].chunk_lens for r in reqs], [0, 0], kg, vg, stride, keep, want_sel=True)
    torch.cuda.synchronize()
    P.cb_destroy(ctx)
    for b, (w, _, _, npl, xn, kpre, vpre) in enumerate(reqs):
        sel = [s.cpu().numpy().astype(np.int64) for s in out.sel[b]]
        ref = O.fuse_prefill(xn, npl, model, w.chunk_lens, 0, kpre, vpre, keep[b], forced_sel=sel,
                             kv_round=O.storage_round("bf16"))
        for l in range(3):
            rows = slice(b * stride, b * stride + w.n_ctx)
            assert max_abs_rel(to_np(kg[l][rows].cpu()), ref.K[l]) < TOL["bf16"], (b, l)
            assert max_abs_rel(to_np(vg[l][rows].cpu()), ref.V[l]) < TOL["bf16"], (b, l)
