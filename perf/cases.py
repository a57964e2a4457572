"""Timing cases of the fusing path: what a serving program has the library do, through its public entry points.

    op            one pass
    request       the chunks' caches are laid into the request's cache, then cb_fuse_prefill
    batched       the same for several requests stacked in one cb_fuse_prefill_batched call
    pipelined     cb_fuse_prefill_pipelined: the chunks' caches come from pinned host memory
    layer         one selective layer, cb_fuse_layer with a check (a program that walks the layers itself)
    chunk         producer.chunk_prefill: the pre-computation of one chunk's cache
    first_token   cb_first_token on the last query row

The fusing calls update the caches in place, so a pass begins by laying the pre-computed rows into them: one copy,
which a program that keeps its chunk caches in device memory makes as well.  Models are those of workloads/configs.py at
their real widths; the two large ones run with fewer layers (every layer is the same work, and a state has to leave room
for others on the card).

The random weights are scaled the way decoders are initialised: every projection has unit gain (standard deviation
1/sqrt(inputs)), the two that feed the residual stream a tenth of it (1/sqrt(2 x 50 layers)).  A layer then adds to the
residual stream without amplifying rounding errors, and scores stay of order one, so that a tie between two tokens in
the selection, decided by the last bit of a sum, changes the fused cache by little.
"""
import random
from dataclasses import replace
from types import SimpleNamespace

import torch

import paper_2405_16444_amd as P
from paper_2405_16444_amd import producer
from workloads import synth
from workloads.configs import LLAMA_70B, MISTRAL_7B, TINY, YI_34B

MODELS = {"tiny": TINY, "mistral7b": MISTRAL_7B, "yi34b": YI_34B, "llama70b": LLAMA_70B}


def _case(op, model, layers=1, chunks=1, shortest=512, longest=512, suffix=64, ratio=0.15, flat=False,
          rope="adjacent", weights="native", requests=1, name=None):
    """chunks lengths in [shortest, longest] per request; ratio: average share of the context tokens recomputed."""
    c = {"name": name} if name else {}
    c.update(op=op, model=model, layers=layers, chunks=chunks, shortest=shortest, longest=longest, suffix=suffix,
             ratio=ratio, flat=flat, rope=rope, weights=weights, requests=requests)
    return c


def listed():
    return [
        # a float model with a few hundred tokens: the smallest request, bound by latency and launches
        _case("request", "tiny", 2, 4, 128, 128, 32, name="tiny_request"),
        # three short passages of odd lengths in front of a short question
        _case("request", "mistral7b", 32, 3, 60, 260, 21, name="short_request"),
        # the usual retrieval request: six chunks of 512 tokens
        _case("request", "mistral7b", 32, 6, 512, 512, 64, name="usual_request"),
        # a larger model at the lowest recompute ratio: few rows against every weight
        _case("request", "yi34b", 20, 6, 512, 512, 64, 0.05, name="low_ratio_request"),
        # the largest model, ten chunks of 400 tokens
        _case("request", "llama70b", 20, 10, 400, 400, 64, name="large_model_request"),
        # the same model served with 8-bit weights, chunks of uneven length, heads in the half-split rotary order
        _case("request", "llama70b", 16, 8, 180, 420, 47, rope="half", weights="int8", name="int8_request"),
        # a long context of 32 uneven chunks (about 20 K tokens)
        _case("request", "mistral7b", 32, 32, 256, 1024, 128, name="long_request"),
        # four users' requests of different lengths in one call
        _case("batched", "mistral7b", 16, 5, 150, 640, 40, requests=4, name="batched_requests"),
        # the chunks' caches are fetched from host memory while layers are recomputed, one ratio for all layers
        _case("pipelined", "yi34b", 12, 6, 300, 512, 64, flat=True, name="host_loaded_request"),
        # one selective layer called by itself
        _case("layer", "mistral7b", 1, 6, 512, 512, 64, rope="half", name="one_layer"),
        # a new chunk enters the store: its cache is computed alone, every row through every layer
        _case("chunk", "mistral7b", 32, 1, 512, 512, name="chunk_cache"),
        # the first token after the prefill: a vocabulary projection for one row
        _case("first_token", "llama70b", name="first_token"),
    ]


def _log(rng, lo, hi):
    return int(round(lo * (hi / lo) ** rng.random()))


def draw(rng):
    op = rng.choice(["request"] * 5 + ["batched", "batched", "pipelined", "layer", "layer", "chunk", "chunk", "first_token"])
    if op == "first_token":
        # the vocabulary is the model's own; the number of query rows is what varies (the last one is projected)
        return _case(op, rng.choice(["mistral7b", "yi34b", "llama70b"]), suffix=rng.randint(1, 512))
    model = rng.choice(["tiny", "mistral7b", "mistral7b", "yi34b", "llama70b"] if op in ("request", "chunk")
                       else ["mistral7b", "mistral7b", "yi34b", "llama70b"])
    rope = rng.choice(["adjacent", "adjacent", "half"])
    weights = rng.choice(["native", "native", "native", "int8"]) if model != "tiny" else "native"
    layers = {"tiny": 2, "mistral7b": rng.randint(8, 32), "yi34b": rng.randint(4, 16), "llama70b": rng.randint(4, 14)}[model]
    if op == "chunk":
        n = _log(rng, 16, 2048)
        return _case(op, model, layers, 1, n, n, rope=rope, weights=weights)
    if op == "layer":
        layers = 1
    requests = rng.randint(2, 6) if op == "batched" else 1
    # context tokens of a request: at most about 20 K, fewer where several share a call or the model is large
    most = {"tiny": 2048, "mistral7b": 16384, "yi34b": 6144, "llama70b": 6144}[model] // requests
    longest = _log(rng, 40, 1024)
    chunks = max(2, min(32, _log(rng, 100, most) // longest))
    return _case(op, model, layers, chunks, rng.randint(max(1, longest // 3), longest), longest, _log(rng, 1, 128),
                 rng.choice([0.05, 0.1, 0.15, 0.15, 0.2, 0.3]), rng.random() < 0.25, rope, weights, requests)


def _shape(case):
    """(model shape, per request its chunk lengths, per request its keep counts)"""
    m = replace(MODELS[case["model"]], n_layers=case["layers"], rope_layout=case["rope"], weight_format=case["weights"])
    rng = random.Random(repr(sorted((k, v) for k, v in case.items() if k != "name")))
    lens = [[rng.randint(case["shortest"], case["longest"]) for _ in range(case["chunks"])]
            for _ in range(case["requests"])]
    keep = [P.cb_default_schedule(m.n_layers, sum(cl), case["ratio"], 0.0, case["flat"]) for cl in lens]
    return m, lens, keep


def _layer_rows(case, lens):
    """(candidates, kept) of the layer op: the second selective layer of a deep model, gradual schedule"""
    keep = P.cb_default_schedule(32, sum(lens), case["ratio"], 0.0, case["flat"])
    return keep[1], keep[2]


def _weights(m, seed):
    layers = []
    for l in range(m.n_layers):
        lw = synth.layer_weights(m, l, seed, device="cuda")
        for name, w in lw.items():
            if name.startswith("w"):
                w *= (0.1 if name in ("wo", "w_down") else 1.0) * w.shape[1] ** -0.5 / synth.WEIGHT_STD
        layers.append(synth.quantize_int8(lw) if m.weight_format == "int8" else lw)
    return layers


def _caches(m, n_rows):
    """K and V caches of every layer in one allocation: [2, layers, rows, kv heads, head_dim]"""
    return torch.zeros((2, m.n_layers, n_rows, m.n_kv_heads, m.head_dim), dtype=synth.storage_dtype(m), device="cuda")


def _precompute(ctx, layers, x, lens, cache, row0, n_rows):
    ks, vs = producer.chunk_prefill(ctx, layers, x, lens, n_rows)
    for l in range(len(layers)):
        cache[0, l, row0:row0 + n_rows] = ks[l]
        cache[1, l, row0:row0 + n_rows] = vs[l]


def prepare(case, seed):
    m, lens, keep = _shape(case)
    op, S, dt = case["op"], case["suffix"], synth.storage_dtype(m)
    s = SimpleNamespace(op=op, model=m, lens=lens, keep=keep, S=S)
    if op == "first_token":
        head = synth.head_weights(m, seed, device="cuda")
        s.norm, s.lm_head = head["final_norm"], head["lm_head"]
        s.hidden = synth.random_rows(S, m.d_model, 2.0, seed + 1, device="cuda")
        s.ctx = P.cb_create(m, S)
        s.logits = torch.empty(m.vocab, dtype=torch.float32, device="cuda")
        s.token = torch.empty(1, dtype=torch.int32, device="cuda")
        return s
    s.layers = _weights(m, seed)
    C = [sum(cl) for cl in lens]
    T = [c + S for c in C]
    stride = max(T)
    s.ctx = P.cb_create(m, stride)
    s.x = synth.random_rows(sum(T), m.d_model, 1.0, seed + 7, device="cuda", dtype=dt)
    if op == "chunk":
        return s
    if op == "layer":
        # Candidates spread over the context, and a cache in which the k to be kept stand out: the deviation
        # of trained models is concentrated in a small share of the tokens (the premise of the method).
        n_cand, s.k = _layer_rows(case, lens[0])
        g = torch.Generator(device="cuda")
        g.manual_seed(seed + 11)
        ctx_pos = torch.randperm(C[0], generator=g, device="cuda")[:n_cand].sort().values
        s.pos = torch.cat([ctx_pos, torch.arange(C[0], T[0], device="cuda")]).to(torch.int32)
        s.h = synth.random_rows(n_cand + S, m.d_model, 1.0, seed + 13, device="cuda")
        s.pre, s.cache = _caches(m, T[0]), _caches(m, T[0])
        s.pre.copy_(synth.random_rows(2 * T[0], m.kv_dim, 1.0, seed + 17, device="cuda").view(s.pre.shape))
        s.ws = torch.empty(P.cb_layer_workspace_bytes(s.ctx, n_cand + S), dtype=torch.uint8, device="cuda")
        s.cache.copy_(s.pre)
        fresh = s.cache[:, 0]
        P.cb_fuse_layer(s.ctx, 0, s.layers[0], s.h, s.pos, S, fresh[0], fresh[1], n_cand, workspace=s.ws)
        rows = ctx_pos
        noise = synth.random_rows(2 * n_cand, m.kv_dim, 1.0, seed + 19, device="cuda")
        noise = noise.view(2, n_cand, m.n_kv_heads, m.head_dim)
        high = torch.zeros(n_cand, device="cuda")
        high[torch.randperm(n_cand, generator=g, device="cuda")[:s.k]] = 1.0
        size = (0.1 + 0.4 * high) * (1.0 + 0.3 * torch.rand(n_cand, generator=g, device="cuda"))
        s.pre[:, 0, rows] = (fresh[:, rows].float() + size[None, :, None, None] * noise).to(dt)
        return s
    s.structs = None
    n_rows = stride * len(lens) if op == "batched" else T[0]
    s.cache = _caches(m, n_rows)
    s.pre = torch.empty_like(s.cache)
    o = 0
    for b, cl in enumerate(lens):
        row0 = b * stride if op == "batched" else 0
        _precompute(s.ctx, s.layers, s.x[o:o + C[b]], cl, s.pre, row0, stride if op == "batched" else T[b])
        o += T[b]
    s.k, s.v = list(s.cache[0]), list(s.cache[1])
    s.stride, s.out = stride, None
    if op == "batched":
        s.ws = torch.empty(P.cb_batched_workspace_bytes(s.ctx, sum(T)), dtype=torch.uint8, device="cuda")
    else:
        s.ws = torch.empty(P.cb_prefill_workspace_bytes(s.ctx, T[0]), dtype=torch.uint8, device="cuda")
    if op == "pipelined":
        host = torch.empty((2, m.n_layers, C[0], m.n_kv_heads, m.head_dim), dtype=dt, pin_memory=True)
        host.copy_(s.pre[:, :, :C[0]])
        s.pre = None
        s.hk, s.hv, s.copy_stream = list(host[0]), list(host[1]), torch.cuda.Stream()
    torch.cuda.synchronize()
    return s


def run(s):
    if s.op == "first_token":
        return P.cb_first_token(s.ctx, s.hidden, s.norm, s.lm_head, logits=s.logits, token=s.token)
    if s.op == "chunk":
        return producer.chunk_prefill(s.ctx, s.layers, s.x[:sum(s.lens[0])], s.lens[0], sum(s.lens[0]))
    if s.op == "layer":
        s.cache.copy_(s.pre)
        h, pos, dev = P.cb_fuse_layer(s.ctx, 0, s.layers[0], s.h, s.pos, s.S, s.cache[0, 0], s.cache[1, 0], s.k,
                                      want_dev=True, workspace=s.ws)
        return h, pos, dev, s.cache
    if s.op == "pipelined":
        s.out = P.cb_fuse_prefill_pipelined(s.ctx, s.layers, s.x, s.lens[0], s.S, s.hk, s.hv, s.k, s.v, s.keep[0],
                                            s.copy_stream, workspace=s.ws, weight_structs=s.structs, out=s.out)
    elif s.op == "batched":
        s.cache.copy_(s.pre)
        s.out = P.cb_fuse_prefill_batched(s.ctx, s.layers, s.x, s.lens, [s.S] * len(s.lens), s.k, s.v, s.stride, s.keep,
                                          workspace=s.ws, weight_structs=s.structs, out=s.out)
    else:
        s.cache.copy_(s.pre)
        s.out = P.cb_fuse_prefill(s.ctx, s.layers, s.x, s.lens[0], s.S, s.k, s.v, s.keep[0], workspace=s.ws,
                                  weight_structs=s.structs, out=s.out)
    s.structs = s.out.weight_structs
    return s.out.final_hidden, s.cache


def _layer_flops(m, n_in, n_kept, positions):
    """positions: sum over the kept rows of (position + 1)"""
    d, q, kv = m.d_model, m.q_dim, m.kv_dim
    return 2.0 * n_in * d * 2 * kv + n_kept * (4.0 * d * q + 6.0 * d * m.d_ff) + 4.0 * q * positions


def work(case):
    m, lens, keep = _shape(case)
    op, S, es = case["op"], case["suffix"], 4 if case["model"] == "tiny" else 2
    if op == "first_token":
        return {"bytes": m.vocab * m.d_model * es + m.vocab * 4 + m.d_model * 4, "flops": 2.0 * m.vocab * m.d_model}
    weights = m.n_layers * m.params_per_layer * (1 if m.weight_format == "int8" else es)
    row = 2 * m.kv_dim * es                                 # K and V of one token on one layer
    flops = moved = 0.0
    for cl, kc in zip(lens, keep):
        C = sum(cl)
        if op == "chunk":
            flops += m.n_layers * _layer_flops(m, C, C, C * (C + 1) / 2)
            moved += C * (m.d_model * es + m.n_layers * row)
            continue
        suffix = S * (C + (S + 1) / 2)                      # sum of (position + 1) over the query rows
        if op == "layer":
            n, k = _layer_rows(case, cl)
            flops += _layer_flops(m, n + S, k + S, k * C / 2 + suffix)
            # the cache is laid out (read and written) and read, kept rows are written
            moved += (n + k + 2 * S) * m.d_model * 4 + C * row * 2 + C * row + (k + S) * row
            continue
        n = C + S
        moved += n * m.d_model * es + S * m.d_model * 4
        for k in kc:
            flops += _layer_flops(m, n, k + S, k * C / 2 + suffix)
            # reused rows are laid out (read and written), re-aligned, and read by attention; kept rows are written
            moved += C * row * 2 + (C + S) * row + (k + S) * row
            n = k + S
    return {"bytes": weights + moved, "flops": flops}


def tolerance(case):
    """Measured with the projections' sums split otherwise along K and the keys cut into other pieces: bf16 caches and
    hidden states move by 0.0014 .. 0.0024 (0.006 where a tie in the selection moved one of few rows; a row that is
    recomputed on one side and reused on the other moves single elements by up to 0.8 of the root mean square)."""
    if case["op"] == "first_token":
        return {"rel": 1e-4}      # one rounding of the normalised row to bf16 that falls the other way: 4e-5
    if case["model"] == "tiny":
        return {"rel": 1e-5}      # float sums in another order
    return {"rel": 1e-2, "max": 0.95}
