"""dK/dV at head dimension 64 with the query tiles of a key tile split over two groups of waves: one, two and three
tiles (the second group has none, or fewer than the first), the diagonal in one or both groups, ragged ends, and
grids on both sides of the rule."""
import pytest

from oracle import attention_ref as A
from paper_2507_00394_amd import inputs as I

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("H,S,causal", [
    (1, 1, True), (2, 64, True), (1, 65, True), (2, 129, True), (1, 192, True), (2, 200, True), (3, 320, True), (1, 1000, True),
    (171, 321, True), (170, 321, True), (4, 1023, False), (4, 1024, False), (1, 1089, False), (28, 1100, False), (29, 1100, False),
    (48, 1030, True), (32, 2100, True),
])
def test_dkdv(H, S, causal):
    from tests import gpu_util as G

    cfg, bits = I.random_case_bits(9500 + S + H, 1, H, S, 64)
    out = G.run_fwd_bwd(bits, cfg.scale, causal)
    heads = list(range(H)) if H < 10 else [0, H // 2, H - 1]
    x = {t: I.bf16_bits_to_float(bits[t][:, heads]) for t in bits}
    ref = A.attn_bwd_ref(x["q"], x["k"], x["v"], x["dO"], cfg.scale, causal)
    for n in ("dk", "dv"):
        assert bool(out[n].isfinite().all()), n
        G.check(n, G.to_f64(out[n][:, heads].contiguous()), ref[n])
