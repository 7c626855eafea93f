"""dK/dV at head dimension 64 with the query tiles of a key tile split over two groups of waves: one, two and three
tiles (the second group has none, or fewer than the first), the diagonal in one or both groups, ragged ends, and
grids on both sides of the rule.  Few heads take groups of two waves on 64 keys; the second test asserts which variant it runs."""
import pytest

from oracle import attention_ref as A
from paper_2507_00394_amd import inputs as I
from tests.dispatch_host import ask

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


TOGETHER_128, SEPARATE = (3,), (0, 1)   # two groups of four waves on 128 keys; one group


@pytest.mark.parametrize("kinds,H,S,causal", [
    (TOGETHER_128, 77, 65, True), (TOGETHER_128, 56, 129, True), (TOGETHER_128, 56, 192, True), (TOGETHER_128, 46, 200, True), (TOGETHER_128, 38, 320, True),
    (TOGETHER_128, 18, 1000, True), (TOGETHER_128, 11, 1023, False), (TOGETHER_128, 11, 1024, False), (TOGETHER_128, 10, 1089, False),
    (SEPARATE, 185, 129, True), (SEPARATE, 200, 192, True), (SEPARATE, 72, 1000, True), (SEPARATE, 52, 1023, False), (SEPARATE, 45, 1089, False)])
def test_dkdv_of_wide_key_tiles(kinds, H, S, causal):
    assert ask([(64, H, S, causal)], "gradient_tiles(D, BH, S, causal)")[0][0] in kinds
    test_dkdv(H, S, causal)
