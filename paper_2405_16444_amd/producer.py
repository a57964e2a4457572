"""Producer of the pre-computed chunk caches KV^pre (paper Sec. 4.1): every chunk is
prefilled alone at positions 0.. .  This is the step *before* the fusing path and is
not part of a request's time.  A chunk is a fusing pass of its own that keeps every row and has no query
rows: one cb_fuse_prefill call, which leaves out the part of the last layer that no key or value depends on."""
from __future__ import annotations

from typing import Dict, Sequence

import torch

from . import binding as B


def chunk_prefill(ctx: B.Context, layers: Sequence[Dict[str, torch.Tensor]], x_ctx: torch.Tensor,
                  chunk_lens: Sequence[int], n_rows_alloc: int):
    """Returns (k_layers, v_layers): per layer a [n_rows_alloc, Hkv, dh] tensor whose
    rows [0, sum(chunk_lens)) hold the chunks' K/V as cached at positions 0.. ."""
    m = ctx.model
    layers = [layers[l] for l in range(m.n_layers)]        # anything indexable; entries past the model's are not looked at
    n_ctx = sum(chunk_lens)
    # a tensor of its own for every layer's K and V: each can be kept, saved or freed without the others.  The chunks fill
    # rows [0, n_ctx), only the rest has to be cleared.
    shape = (n_rows_alloc, m.n_kv_heads, m.head_dim)
    ks = [torch.empty(shape, dtype=ctx.dtype, device=ctx.device) for _ in range(m.n_layers)]
    vs = [torch.empty(shape, dtype=ctx.dtype, device=ctx.device) for _ in range(m.n_layers)]
    if n_rows_alloc > n_ctx:
        torch._foreach_zero_([t[n_ctx:] for t in ks + vs])
    ws = torch.empty(B.cb_prefill_workspace_bytes(ctx, max(chunk_lens)), dtype=torch.uint8, device=ctx.device)
    structs, o = None, 0
    for ln in chunk_lens:
        # the chunk's cache rows are a contiguous slice, addressed as a cache of ln tokens
        kc, vc = [k[o:o + ln] for k in ks], [v[o:o + ln] for v in vs]
        x = x_ctx[o:o + ln]
        o += ln
        if x.dtype == ctx.dtype:
            x = x.contiguous()
            if x.dtype != torch.float32 and x.data_ptr() % 16:
                x = x.clone()               # 16-bit rows may start anywhere (a float input is read where it lies, below too)
            out = B.cb_fuse_prefill(ctx, layers, x, [ln], 0, kc, vc, [ln] * m.n_layers, workspace=ws,
                                    weight_structs=structs)
            structs = out.weight_structs
            continue
        # an input of another precision than the model's storage type is not rounded to it: layer by layer
        h = x.to(torch.float32).contiguous()
        pos = torch.arange(ln, dtype=torch.int32, device=ctx.device)
        for l in range(m.n_layers):
            h, _, _ = B.cb_fuse_layer(ctx, l, layers[l], h, pos, 0, kc[l], vc[l], ln, workspace=ws)
    return ks, vs
