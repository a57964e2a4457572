"""The software-pipelined attention kernel where it can go wrong: key counts around the edges of its 32-key
sub-tiles and 64-key tiles (one sub-tile, an odd and an even number, the ring of four tiles once and more than
once around), rows whose last key lies in each of them, and scores that keep rising along the keys, so that the
running maximum has to move late although it is allowed to lag behind by a factor 2^8."""
import numpy as np
import pytest
import torch

from oracle import cacheblend_oracle as O
from workloads.configs import ModelShape

from gpu_util import TOL, announce, max_abs_rel, to_np
from test_gpu_parity import layer_case, oracle_layer, run_layer_both

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def P():
    import paper_2405_16444_amd as pkg
    return pkg


@pytest.mark.parametrize("dh,hq,hkv", [(64, 4, 2), (128, 4, 1)])
@pytest.mark.parametrize("n_tokens", [1, 31, 32, 33, 64, 65, 96, 97, 128, 191, 256, 257, 320, 449])
def test_every_row_of_short_caches(P, n_tokens, dh, hq, hkv):
    model = ModelShape(1, 256, hq, hkv, dh, 512, 1e-5, 1e4, "bf16")
    announce("attention over a short cache", n_tokens, dh)
    lw, h, pos, kc, vc = layer_case(model, n_tokens, n_tokens, 0, seed=700 + n_tokens)
    h_out, pos_out, _, kg, vg = run_layer_both(P, model, lw, h, pos, kc, vc, 0, n_tokens, want_dev=False)
    h_ref, pos_ref, _, _, _ = oracle_layer(model, lw, h, pos, kc, vc, 0, n_tokens, None)
    assert np.array_equal(pos_out.numpy(), pos_ref)
    assert max_abs_rel(to_np(h_out), h_ref) < TOL["bf16"]


@pytest.mark.parametrize("dh,hq,hkv", [(64, 4, 2), (128, 4, 1)])
@pytest.mark.parametrize("n_tokens,n_rows", [(200, 5), (700, 90), (2100, 40), (1500, 600)])
def test_scores_that_rise_along_the_keys(P, n_tokens, n_rows, dh, hq, hkv):
    """The cached keys grow with their position by a factor 60: the largest score of a row moves by far more than
    the slack between early and late tiles, in either direction for half of the rows.  Scores reach about 12, so the
    rounding of a query to bf16 (2^-9) moves a probability by 12/512 = 2.3 %, of an attention output that is a few
    per cent of the residual stream: well inside the usual bound."""
    model = ModelShape(1, 256, hq, hkv, dh, 512, 1e-5, 1e4, "bf16")
    announce("rising scores", n_tokens, n_rows, dh)
    lw, h, pos, kc, vc = layer_case(model, n_tokens, n_rows, 4, seed=900 + n_rows)
    ramp = torch.logspace(-1.3, 0.48, n_tokens).view(-1, 1, 1)
    kc = (kc.float() * ramp / kc.float().square().mean().sqrt()).to(kc.dtype)
    h_out, pos_out, _, kg, vg = run_layer_both(P, model, lw, h, pos, kc, vc, 4, n_rows - 4, want_dev=False)
    h_ref, _, _, _, _ = oracle_layer(model, lw, h, pos, kc, vc, 4, n_rows - 4, None)
    assert bool(torch.isfinite(h_out).all())
    assert max_abs_rel(to_np(h_out), h_ref) < TOL["bf16"]
