"""Models whose shared network has layers, or whose anchor network has none (GPU).

With shared layers the embedding gather writes c alone and the copies and norms that follow it
run on their own; without anchor layers it writes the anchor states and no norm.  A refresh
and a stale step, with and without a prefilled context and a self-conditioning signal, against
the float64 oracle at the bars of the other step tests.  Each part is held to its bar on the
GPU's own input: the fusion's closing LayerNorm takes states of rms 0.076 to rms 1, and with
them the earlier layers' bf16 rounding (rms 0.0004) 13-fold, to where a chained comparison's
largest of 18 944 errors passes 2e-2 with no error in the fusion.
"""
import numpy as np
import pytest
import torch

import paper_2609_37924_amd as tadm
import synth
from helpers import dev, gpu_model, oracle_net, rows_close

pytestmark = pytest.mark.gpu

TINY = dict(base="tiny", n_shared=1)
SMALL = dict(base="small", d_model=512, n_heads=8, n_kv_heads=8, d_ffn=1024, vocab=1024, n_shared=1, n_anchor=1, n_denoise=1)
PAIRED = dict(fusion_kind="paired")


@pytest.mark.parametrize("over", [
    TINY, dict(TINY, n_shared=2, n_anchor=0), dict(TINY, n_shared=0, n_anchor=0), dict(TINY, n_denoise=0),
    dict(TINY, fusion_rank=32, **PAIRED), dict(TINY, n_shared=0, n_anchor=0, fusion_rank=32, **PAIRED),
    SMALL, dict(SMALL, n_anchor=0), dict(SMALL, n_shared=0, n_anchor=0), dict(SMALL, fusion_rank=256, **PAIRED)])
@pytest.mark.parametrize("P", [0, 21])
def test_shared_layers(over, P):
    over = dict(over)
    cfg = synth.get_config(over.pop("base"), **over)
    tol = dict(rtol=1e-4, atol=1e-4) if cfg["dtype"] == "f32" else dict(rtol=2e-2, atol=2e-2)
    B, L, off, d, V = 2, 37, 5, cfg["d_model"], cfg["vocab"]
    Lc = L - off
    g = torch.Generator().manual_seed(9)
    z0, z1 = (torch.randint(0, V + 1, (B, L), generator=g, dtype=torch.int32) for _ in range(2))
    prompt = torch.randint(0, V, (B, max(P, 1)), generator=g, dtype=torch.int32)
    sc0, sc1 = (0.02 * torch.randn(B, Lc, d, generator=g) for _ in range(2))
    tensors = synth.make_weights(cfg, perturb=True)
    net = oracle_net(cfg, tensors)
    m = gpu_model(cfg, tensors, B, P + L)
    try:
        tadm.tadm_debug_taps(m, 1)
        ctx = None
        if P:
            ctx = tadm.tadm_context_create(m, B, P + L)
            tadm.tadm_context_append(m, ctx, prompt.to(dev()), B, P)
        cache = tadm.tadm_cache_create(m, B, L)
        d0, d1, s0, s1 = z0.to(dev()), z1.to(dev()), sc0.to(dev()), sc1.to(dev())
        got = {}
        for sc in (False, True):
            if sc:
                tadm.tadm_anchor_forward_sc(m, ctx, d0, B, L, 8, 8, s0, off, cache)
                args = tadm.step_args(6, 8, 0, 2, 4, 1.0, entropy_eta=0.2, sc_in=s1)
            else:
                tadm.tadm_anchor_forward(m, ctx, d0, B, L, 8, 8, cache)
                args = tadm.step_args(6, 8, 3, 2, 4, 1.0)
            logits = torch.empty(B, Lc, V, device=dev())
            nxt = torch.empty_like(d1)
            tadm.tadm_denoise_step(m, ctx, d1, B, L, off, cache, args, logits, nxt)
            c, h, ch, ht = (torch.empty(B, L, d, device=dev()) for _ in range(4))
            tadm.tadm_debug_read(m, tadm.TAP_EMBED, c)
            tadm.tadm_debug_read(m, tadm.TAP_FUSED, ht)
            tadm.tadm_cache_read(cache, tadm.CACHE_H, h)
            tadm.tadm_cache_read(cache, tadm.CACHE_C, ch)
            torch.cuda.synchronize()
            got[sc] = [t.cpu().numpy() for t in (ch, h, c, ht, logits)]
        pos = np.arange(P, P + L)
        for b in range(B):
            kv = net.fresh_kv(prompt[b].numpy(), np.arange(P)) if P else None
            for sc in (False, True):
                pad = [np.concatenate([np.zeros((off, d)), s[b].double().numpy()]) if sc else None for s in (sc0, sc1)]
                ch, h, c, ht, logits = (x[b].astype(np.float64) for x in got[sc])
                for what, x, ref in (("anchor c", ch, net.shared(z0[b].numpy(), pos, kv, sc=pad[0])),
                                     ("anchor h", h, net.anchor_cache(ch, pos, kv)["h"]),
                                     ("c", c, net.shared(z1[b].numpy(), pos, kv, sc=pad[1])),
                                     ("fused", ht, net.fuse(c, {"h": h, "c": ch})),
                                     ("logits", logits, net.head(net.denoise(ht, pos, kv)[off:]))):
                    rows_close(x, ref, what=f"{what} row {b} sc {sc}", **tol)
        tadm.tadm_cache_destroy(cache)
        if ctx is not None:
            tadm.tadm_context_destroy(ctx)
    finally:
        tadm.tadm_model_destroy(m)
