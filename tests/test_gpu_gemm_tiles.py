"""The matrix products at the edges of their tiles and K tiles.

The vocabulary head of a model without layers is one product of known operands: its
normalised input is read back (bf16, exact as float32) and the logits are compared with the
float64 product of that input and the stored weights.  d_model 64 to 704 gives one
to eleven K tiles; the row counts and vocabularies leave partial tiles of every size that the
dispatch knows and grids with and without an even split over the chip's eight dies.
"""
import pytest
import torch

import synth

pytestmark = pytest.mark.gpu


def _model(d, vocab, B, P, G, base="small", nan_rows=()):
    import paper_2609_37924_amd as tadm
    heads = dict(n_heads=d // 64, n_kv_heads=d // 64, d_ffn=64) if base == "small" else dict(
        n_heads=d // 4, n_kv_heads=d // 4, head_dim=4, d_ffn=16)
    cfg = synth.get_config(base, d_model=d, vocab=vocab, n_anchor=0, n_denoise=0, **heads)
    dev = torch.device("cuda:0")
    tensors = [t.to(dev) for t in synth.make_weights(cfg, perturb=True)]
    tensors[2][list(nan_rows)] = float("nan")  # w_out
    m = tadm.load_model(cfg, tensors, max_batch=B, max_seq=P + G, stream=torch.cuda.current_stream().cuda_stream)
    return tadm, cfg, dev, tensors, m


@pytest.mark.parametrize("d,vocab,B,G", [(128, 32768, 1, 257), (192, 33028, 1, 300), (320, 33028, 3, 100),
                                         (128, 16640, 2, 512), (192, 65540, 1, 63),
                                         (64, 300, 1, 63), (64, 516, 1, 1), (128, 1028, 1, 65), (320, 5000, 1, 129),
                                         (704, 96, 2, 33), (640, 3000, 3, 100),
                                         # 256 x 256 tiles: one and two per block, two to eleven K tiles
                                         (192, 3836, 4, 1025), (128, 6396, 4, 1250), (704, 6396, 4, 1250),
                                         # the same tiles, a block each (short K, fewer than 4 096 rows)
                                         (192, 32764, 2, 250), (128, 16388, 3, 1333),
                                         # 192 x 128 tiles above and below 4 096 rows, 64 x 64 at three and more per CU, 64 x 96
                                         (192, 2300, 4, 1030), (128, 9000, 2, 500), (192, 3900, 1, 900),
                                         (320, 1028, 2, 1040)])
def test_product_tiles(d, vocab, B, G):
    _head_product(*_model(d, vocab, B, 1, G), d, vocab, B, G)


@pytest.mark.parametrize("d,vocab,B,G", [(4, 4, 1, 1), (20, 12, 1, 17), (36, 100, 2, 15), (64, 256, 1, 24),
                                         (132, 1028, 1, 33), (260, 516, 3, 16), (64, 4096, 1, 257),
                                         (132, 2052, 3, 100)])
def test_float32_product_tiles(d, vocab, B, G):
    """float32 models: small products (16 x 16 tiles, K split over four waves, K not a multiple
    of 16) and two beyond them (64 x 64 tiles, up to 2 048 tiles of 16 x 16 on the former)."""
    _head_product(*_model(d, vocab, B, 1, G, base="tiny"), d, vocab, B, G)


@pytest.mark.parametrize("d,F,vocab,B,L", [(64, 256, 4096, 32, 17), (132, 272, 1028, 130, 33), (256, 1024, 512, 40, 65)])
def test_float32_rows_do_not_depend_on_the_batch(d, F, vocab, B, L):
    """A float32 row has the same bits alone and in a batch whose products (layers, fusion, head)
    are large enough for the other kernel: its anchor states, its logits, and the tokens and
    confidences of a masked-only step, whose head has a row bound of the whole batch."""
    import paper_2609_37924_amd as tadm
    cfg = synth.get_config("tiny", d_model=d, vocab=vocab, n_heads=d // 4, n_kv_heads=d // 4, head_dim=4, d_ffn=F,
                           n_anchor=1, n_denoise=1)
    dev = torch.device("cuda:0")
    m = tadm.load_model(cfg, [t.to(dev) for t in synth.make_weights(cfg, perturb=True)], max_batch=B, max_seq=L,
                        stream=torch.cuda.current_stream().cuda_stream)
    try:
        z = torch.randint(0, vocab, (B, L), generator=torch.Generator().manual_seed(5), dtype=torch.int32)
        z[:, 1::2] = vocab
        z = z.to(dev)

        def step(b, full):
            cache = tadm.tadm_cache_create(m, b, L)
            zb = z[:b].contiguous()
            tadm.tadm_anchor_forward(m, None, zb, b, L, 1, 1, cache)
            h = torch.empty(b, L, d, device=dev)
            tadm.tadm_cache_read(cache, tadm.CACHE_H, h)
            logits = torch.empty(b, L - 1, vocab, device=dev) if full else None
            nxt = torch.empty_like(zb)
            tadm.tadm_denoise_step(m, None, zb, b, L, 1, cache, tadm.step_args(1, 1, L // 4, 2, 11, 1.0), logits, nxt)
            ch = torch.empty(b, L - 1, dtype=torch.int32, device=dev)
            cf = torch.empty(b, L - 1, device=dev)
            tadm.tadm_debug_read(m, tadm.TAP_CHOICE, ch)
            tadm.tadm_debug_read(m, tadm.TAP_CONF, cf)
            torch.cuda.synchronize()
            tadm.tadm_cache_destroy(cache)
            out = dict(h=h[0], choice=ch[0], conf=cf[0], next=nxt[0])
            return dict(out, logits=logits[0]) if full else out

        alone = step(1, True)
        for full in (True, False):
            for name, x in step(B, full).items():
                assert torch.equal(x, alone[name]), (name, full)
    finally:
        tadm.tadm_model_destroy(m)


def _head_product(tadm, cfg, dev, tensors, m, d, vocab, B, G):
    try:
        L = G + 1
        z = torch.randint(0, vocab, (B, L), dtype=torch.int32).to(dev)
        cache = tadm.tadm_cache_create(m, B, L)
        tadm.tadm_anchor_forward(m, None, z, B, L, 1, 1, cache)
        logits = torch.full((B, G, vocab), float("nan"), device=dev)
        nxt = torch.empty_like(z)
        tadm.tadm_denoise_step(m, None, z, B, L, 1, cache, tadm.step_args(1, 1, 0, 0, 3, 1.0), logits, nxt)
        x = torch.empty(B, G, d, device=dev)
        tadm.tadm_debug_read(m, tadm.TAP_FINAL, x)
        torch.cuda.synchronize()
        w = tensors[2].double()
        ref = x.double().reshape(-1, d) @ w.T
        # float32 accumulation of d exact products: at most d roundings of 2^-24 of the sum of magnitudes
        bound = d * 2.0 ** -24 * (x.double().abs().reshape(-1, d) @ w.abs().T)
        assert ((logits.double().reshape(-1, vocab) - ref).abs() <= bound).all()
        tadm.tadm_cache_destroy(cache)
    finally:
        tadm.tadm_model_destroy(m)


@pytest.mark.parametrize("d,vocab,B,G,masked", [
    (192, 32768, 4, 256, 3), (192, 40960, 4, 256, 129), (192, 40964, 5, 250, 250), (192, 65536, 2, 700, 0),
    (64, 40960, 1, 256, 256), (128, 41000, 3, 86, 86), (256, 40960, 1, 300, 1), (320, 40100, 2, 260, 65),
    (448, 65540, 1, 129, 129)])
def test_masked_only_head_with_few_rows(d, vocab, B, G, masked):
    """The masked-only head, whose row count is known on the device alone, against the sampler
    on the logits of every row: the same tokens and confidences at any share of masked rows
    (the first `masked` positions of each row; a row bound of all positions)."""
    _masked_only_head(d, vocab, B, G, masked)


@pytest.mark.parametrize("d,vocab,B,G,masked", [(128, 32768, 1, 40, 40), (64, 40960, 2, 70, 33)])
def test_masked_only_head_with_nan_logits(d, vocab, B, G, masked):
    """The same where some vocabulary entries have a NaN logit in every row (NaN weights): alone in
    a normaliser group, several in one, next to each other and 16 apart."""
    _masked_only_head(d, vocab, B, G, masked, nan_rows=[5, 640, 641, 656, 700, vocab - 1])


def _masked_only_head(d, vocab, B, G, masked, nan_rows=()):
    tadm, cfg, dev, tensors, m = _model(d, vocab, B, 1, G, nan_rows=nan_rows)
    try:
        L = G + 1
        z = torch.randint(0, vocab, (B, L), dtype=torch.int32)
        z[:, 1:1 + masked] = vocab
        z = z.to(dev)
        cache = tadm.tadm_cache_create(m, B, L)
        tadm.tadm_anchor_forward(m, None, z, B, L, 1, 1, cache)
        args = tadm.step_args(1, 1, masked, 5, 77, 1.0)
        out = []
        for logits in (torch.empty(B, G, vocab, device=dev), None):
            nxt = torch.empty_like(z)
            ch = torch.empty(B, G, dtype=torch.int32, device=dev)
            cf = torch.empty(B, G, device=dev)
            tadm.tadm_denoise_step(m, None, z, B, L, 1, cache, args, logits, nxt)
            tadm.tadm_debug_read(m, tadm.TAP_CHOICE, ch)
            tadm.tadm_debug_read(m, tadm.TAP_CONF, cf)
            torch.cuda.synchronize()
            out.append((nxt, ch, cf))
        for a, b in zip(*out):
            assert torch.equal(a, b)
        tadm.tadm_cache_destroy(cache)
    finally:
        tadm.tadm_model_destroy(m)


@pytest.mark.parametrize("d,F,B,L", [(128, 192, 1, 1), (128, 1024, 1, 64), (256, 512, 1, 65), (768, 2048, 1, 385),
                                     (128, 8192, 1, 61), (1024, 8192, 1, 128), (1024, 8192, 2, 300),
                                     (1024, 2048, 2, 1037), (768, 512, 1, 1001)])
def test_residual_products(d, F, B, L):
    """Layers whose residual products are whole on 32, 64 and 96-column tiles, or split over K on
    64, 128 and 256-column tiles with the slice sum writing the following norm, against the
    float64 layers of the oracle at the bf16 bar."""
    import numpy as np

    import paper_2609_37924_amd as tadm
    from oracle import network as N

    cfg = synth.get_config("small", d_model=d, n_heads=d // 64, n_kv_heads=d // 64, d_ffn=F, vocab=256, n_anchor=2,
                           n_denoise=0)
    dev = torch.device("cuda:0")
    tensors = synth.make_weights(cfg, perturb=True)
    m = tadm.load_model(cfg, [t.to(dev) for t in tensors], max_batch=B, max_seq=L,
                        stream=torch.cuda.current_stream().cuda_stream)
    try:
        z = torch.randint(0, cfg["vocab"], (B, L), generator=torch.Generator().manual_seed(3), dtype=torch.int32)
        cache = tadm.tadm_cache_create(m, B, L)
        tadm.tadm_anchor_forward(m, None, z.to(dev), B, L, 1, 1, cache)
        h = torch.empty(B, L, d, device=dev)
        tadm.tadm_cache_read(cache, tadm.CACHE_H, h)
        torch.cuda.synchronize()
        net = N.Network(N.Weights(cfg, [s[0] for s in synth.weight_specs(cfg)], tensors))
        pos = np.arange(L)
        for b in range(B):
            ref = net.anchor_cache(net.shared(z[b].numpy(), pos), pos)["h"]
            assert np.allclose(h[b].cpu().numpy(), ref, rtol=2e-2, atol=2e-2)
        tadm.tadm_cache_destroy(cache)
    finally:
        tadm.tadm_model_destroy(m)
