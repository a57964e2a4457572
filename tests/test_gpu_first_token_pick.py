"""The greedy pick of the first-token head, which the workgroups of the vocabulary projection decide among themselves:
vocabularies around the number of rows in flight (16 per workgroup, 4096 in all), ties between rows of different
workgroups (the lower index wins), only negative logits, and several calls on one context in a row."""
import pytest
import torch

from workloads.configs import ModelShape

from gpu_util import announce

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def P():
    import paper_2405_16444_amd as pkg
    return pkg


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("vocab", [1, 15, 16, 17, 255, 4095, 4096, 4097, 9001])
def test_pick_is_the_first_largest_logit(P, dtype, vocab):
    announce("greedy pick", dtype, vocab)
    d, dt = 256, {"bf16": torch.bfloat16, "f32": torch.float32}[dtype]
    g = torch.Generator().manual_seed(vocab)
    w = torch.empty(vocab, d).normal_(0, 0.05, generator=g).to(dt)
    h = torch.empty(3, d).normal_(0, 1, generator=g)
    gain = torch.ones(d, dtype=dt)
    ctx = P.cb_create(ModelShape(1, d, 4, 2, 64, 128, 1e-5, 1e4, dtype, vocab), 8)
    for rep in range(3):
        wr = w.clone()
        if rep > 0:                       # the largest row again at the end and in the middle
            top = int((wr.float() @ h[-1]).argmax())
            wr[vocab - 1] = wr[top]
            wr[vocab // 2] = wr[top]
        if rep == 2:                      # every logit negative: rows against the hidden state
            wr = -(wr.float().abs() * h[-1].sign()).to(dt)
            wr[vocab - 1] = wr[vocab // 2]
        logits, token = P.cb_first_token(ctx, h.cuda(), gain.cuda(), wr.cuda())
        got = logits.cpu()
        # one element of the normalised row may round to bf16 the other way: 2^-6 (values up to 4) x a weight of 0.2
        assert torch.allclose(got, wr.float() @ (h[-1] * torch.rsqrt(h[-1].square().mean() + 1e-5)).to(dt).float(),
                              rtol=1e-3, atol=4e-3)
        assert int(token) == int((got == got.max()).nonzero()[0])
    P.cb_destroy(ctx)


@pytest.mark.parametrize("bits", [0x7FFFFFFF, 0x7FC00000, 0xFFC00000, 0xFFFFFFFF], ids=hex)
@pytest.mark.parametrize("rows", [(0,), (0, 1, 2, 3, 16, 4999), (777,)], ids=str)
def test_nan_logits_lose_and_leave_the_context_usable(P, bits, rows):
    """A NaN logit, whatever its sign and payload, counts as less than every number; the calls that follow on the same
    context are unaffected by it.  (A positive one with every payload bit set used to map row 0 to the value that marks
    the pick's scratch: the token was not written, nor by any later call.)"""
    announce("greedy pick, NaN logits", hex(bits), rows)
    vocab, d = 5000, 256
    g = torch.Generator().manual_seed(5)
    w = torch.empty(vocab, d).normal_(0, 0.05, generator=g)
    bad = w.clone()
    bad.view(torch.int32)[list(rows)] = bits if bits < 2 ** 31 else bits - 2 ** 32
    h, gain = torch.empty(1, d).normal_(0, 1, generator=g).cuda(), torch.ones(d).cuda()
    ctx = P.cb_create(ModelShape(1, d, 4, 2, 64, 128, 1e-5, 1e4, "f32", vocab), 8)
    token = torch.full((1,), -1, dtype=torch.int32, device="cuda")
    for weights, nan_rows in ((bad, rows), (w, ()), (bad, rows), (w, ())):
        token.fill_(-1)
        logits, _ = P.cb_first_token(ctx, h, gain, weights.cuda(), token=token)
        got = logits.cpu()
        assert got.isnan().nonzero().flatten().tolist() == sorted(nan_rows)
        got[list(nan_rows)] = -float("inf")
        assert int(token) == int((got == got.max()).nonzero()[0])
    token.fill_(-1)
    P.cb_first_token(ctx, h, gain, torch.full_like(w, float("nan")).cuda(), token=token)
    assert int(token) == 0
    P.cb_destroy(ctx)
