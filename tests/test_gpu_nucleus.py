"""The nucleus threshold's selection at its limits: rows whose boundary bin holds more weights
than the list in LDS (walked in the row instead), whole rows of one weight, boundaries in
the smallest weights, infinite logits; kept-in-registers and re-read rows, vocabularies that
are not a multiple of four.  Tokens and confidences equal the oracle's bit for bit."""
import numpy as np
import pytest
import torch

import synth
from oracle import sampler as S

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("V,top_p,kind", [
    (40000, 0.5, "close"),       # every weight within 1e-3 of the largest: one bin, no list
    (16384, 0.37, "close"),      # the same in registers
    (40001, 0.5, "close"),       # and with scalar loads
    (50304, 0.9, "equal"),
    (5000, 0.25, "equal"),
    (50304, 0.999, "wide"),      # boundary among the smallest weights
    (32768, 0.9999, "wide"),
    (36004, 0.9, "minus_inf"),   # most of the row excluded
    (4096, 0.6, "plus_minus"),
    (131076, 0.95, "wide"),
])
def test_nucleus_threshold_limits(V, top_p, kind):
    import paper_2609_37924_amd as tadm

    dev, n = torch.device("cuda:0"), 4
    g = torch.Generator().manual_seed(V)
    x = torch.randn(1, n, V, generator=g)
    if kind == "close":
        x = x * 2e-4
    elif kind == "equal":
        x = torch.full_like(x, 0.75)
    elif kind == "wide":
        x = x * 4.0
    elif kind == "minus_inf":
        x[torch.rand(x.shape, generator=g) < 0.95] = -float("inf")
    else:
        x = torch.where(x > 0, torch.full_like(x, 3.0), torch.full_like(x, -20.0))
    cfg = synth.get_config("tiny", vocab=V)
    m = tadm.tadm_model_create(tadm.make_config(cfg, max_batch=1, max_seq=n))
    tadm.tadm_set_stream(m, torch.cuda.current_stream().cuda_stream)
    try:
        tp = float(np.float32(top_p))
        can = torch.full((1, n), V, dtype=torch.int32, device=dev)
        nxt, ch = torch.empty_like(can), torch.empty_like(can)
        cf = torch.empty(1, n, device=dev)
        tadm.tadm_sample(m, x.to(dev), can, 1, n, 0, 9, tadm.step_args(3, 8, n, 6, 77, 1.0, top_p=tp), nxt, ch, cf)
        torch.cuda.synchronize()
        for j in range(n):
            tok, conf = S.sample_position(x[0, j].numpy(), np.float32(1.0), 9 + j, 0, 6, 77, top_p=tp)
            assert ch[0, j].item() == tok
            assert cf[0, j].cpu().numpy().view(np.int32) == np.float32(conf).view(np.int32)
    finally:
        tadm.tadm_model_destroy(m)
