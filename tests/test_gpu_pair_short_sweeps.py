"""Shortest sweeps of the head-dimension-128 dK/dV pass: no, one and few complete 32-row blocks with and without a ragged
last one, around the first step (no mask) and around the four blocks of the diagonal (causal), up to the first
trip of seven blocks whose copies need no check.  Three heads take key tiles of 64 keys; those of 128 have their shortest sweeps in
test_gpu_parity_dkdv_pair.py."""
import pytest

from oracle import attention_ref as A
from paper_2507_00394_amd import inputs as I

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("S,causal", [(s, False) for s in (31, 32, 33, 64, 95, 225, 32 * 13 + 1, 32 * 14)] +
                         [(s, True) for s in (96, 127, 128, 129, 160, 161, 255, 32 * 16, 32 * 17 + 3, 32 * 18)])
def test_dkdv(S, causal):
    from tests import gpu_util as G

    cfg, bits = I.random_case_bits(8800 + S, 1, 3, S, 128)
    out = G.run_fwd_bwd(bits, cfg.scale, causal)
    f = {t: I.bf16_bits_to_float(bits[t]) for t in bits}
    ref = A.attn_bwd_ref(f["q"], f["k"], f["v"], f["dO"], cfg.scale, causal)
    for n in ("dk", "dv"):
        G.check(n, G.to_f64(out[n]), ref[n])
