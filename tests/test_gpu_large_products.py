"""The 256 x 256 product loop's epilogues and second operand at remainders (GPU).

From 4 096 rows on, q/k/v (staged in LDS while the next tile's loads land), the up projection,
the first fusion product (two activation operands), the second and the residual products of a
long K run on 256 x 256 tiles, whose blocks walk several tiles, where these need the fewest
rounds; else on 192 x 128 ones.  9 canvases of 461 positions leave a last tile of 53 rows, and
the odd length puts every 8-token run of V^T at another offset and across the end of a canvas.
On 256 x 256 tiles: q/k/v of 6 144 features (408 tiles, 256 blocks), up projections of 7 552
(510), the fusion products (680 and 136) and FFN down with K = 7 552 (136); q/k/v of 4 096
features and the attention output run on 192 x 128.
"""
import pytest

import synth
from test_gpu_parity import BF16_TOL, _teacher_step_parity

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("over", [dict(n_heads=32, n_kv_heads=32, head_dim=64, ffn_kind="swiglu", d_ffn=3776),
                                  dict(n_heads=16, n_kv_heads=8, head_dim=128, ffn_kind="gelu", d_ffn=7552),
                                  dict(n_heads=16, n_kv_heads=16, head_dim=128, ffn_kind="geglu", d_ffn=3776)])
def test_layers_and_fusion_on_partial_tiles(over):
    cfg = synth.get_config("1b", n_anchor=1, n_denoise=1, vocab=256, prompt_len=0, gen_len=461, **over)
    _teacher_step_parity(cfg, 9, BF16_TOL, rows=[0, 3, 8])
