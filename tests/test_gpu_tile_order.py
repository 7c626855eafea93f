"""The order in which workgroups take the tiles of causal attention: an XCD sweeps its first heads
one after the other and the last ones side by side.  With outputs prefilled with NaN a tile done by nobody
fails the finiteness check, one done under a wrong head the comparison with the oracle."""
import numpy as np
import pytest
import torch

from oracle import attention_ref as A
from paper_2507_00394_amd import inputs as I

pytestmark = pytest.mark.gpu


# (heads, S): 10 heads per XCD of which 4 (1 tile each) to 10 go first; heads shared by 2, 4 and 8 XCDs; at head dimension 128
# three and five tiles of a head to an XCD, of which all but one, all and some go side by side
@pytest.mark.parametrize("BH,S,D", [(80, 2600, 64), (80, 8193, 64), (44, 2600, 64), (42, 1500, 64), (13, 3000, 64), (136, 570, 128), (80, 1100, 128),
                                    (40, 640, 128), (264, 300, 128), (36, 1300, 128), (36, 1200, 128)])
def test_every_tile_once(BH, S, D):
    from tests import gpu_util as G

    cfg, bits = I.random_case_bits(8800 + BH, 1, BH, S, D)
    out = G.run_fwd_bwd(bits, cfg.scale, True)
    for n in ("o", "lse", "dq", "dk", "dv"):
        assert bool(torch.isfinite(out[n].float()).all()), n
    heads = [0, 8, BH // 2, BH - 1]
    x = {t: I.bf16_bits_to_float(bits[t][:, heads]) for t in bits}
    if S > 4000:   # the first rows of O depend on the first keys only
        rows = 1000
        ref = A.attn_bwd_ref(*(x[t][:, :, :rows] for t in ("q", "k", "v", "dO")), cfg.scale, True)
        names = ("o", "dq")
    else:
        rows, names = S, ("o", "dq", "dk", "dv")
        ref = A.attn_bwd_ref(x["q"], x["k"], x["v"], x["dO"], cfg.scale, True)
    for n in names:
        G.check(n, G.to_f64(out[n][:, heads][:, :, :rows].contiguous()), ref[n])
