"""The 256 x 256 product loop's epilogues and second operand at remainders (GPU).

From 4 096 rows on, q/k/v (staged in LDS while the next tile's loads land), the up projection,
the first fusion product (two activation operands), the second and the residual products run
on 256 x 256 tiles, whose blocks walk several tiles.  9 canvases of 461 positions leave
a last tile of 53 rows, and the odd length puts every 8-token run of V^T at another offset and
across the end of a canvas.  Sizes are such that each of these grids has at least 128 tiles
(more than 256 for all but the residual and the second fusion product).
"""
import pytest

import synth
from test_gpu_parity import BF16_TOL, _teacher_step_parity

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("over", [dict(n_heads=32, n_kv_heads=32, head_dim=64, ffn_kind="swiglu", d_ffn=2112),
                                  dict(n_heads=16, n_kv_heads=8, head_dim=128, ffn_kind="gelu", d_ffn=4160),
                                  dict(n_heads=16, n_kv_heads=16, head_dim=128, ffn_kind="geglu", d_ffn=2048)])
def test_layers_and_fusion_on_partial_tiles(over):
    cfg = synth.get_config("1b", n_anchor=1, n_denoise=1, vocab=256, prompt_len=0, gen_len=461, **over)
    _teacher_step_parity(cfg, 9, BF16_TOL, rows=[0, 3, 8])
