"""The backward's dK/dV and dQ passes in one launch or in two: one short tile, ragged ends, the split and the whole query tiles, and
grids on both sides of the line (1024 key tiles at head dimension 128) and of the rule for head dimension 64.  Either way the results equal those of the passes launched one by one, bit for bit, for the work of a workgroup is the
same; and, as separate launches are the same kernels in either call, some heads are held against the oracle."""
import pytest
import torch

from oracle import attention_ref as A
from paper_2507_00394_amd import inputs as I

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("H,S,D,causal", [
    (1, 1, 64, True), (1, 1, 128, False), (3, 129, 64, True), (3, 129, 64, False), (3, 385, 128, True), (2, 640, 128, False),
    (11, 1500, 128, True), (64, 1030, 128, True), (27, 777, 64, False), (128, 511, 64, True), (129, 511, 64, True),
    (512, 129, 128, True), (513, 129, 128, True), (256, 100, 64, False), (257, 100, 64, False),
    # head dimension 64: one launch and two, causal and not, up to grids that fill the chip several times
    (48, 1030, 64, True), (56, 1030, 64, True), (64, 1030, 64, True), (32, 2100, 64, True), (80, 640, 64, False), (24, 1500, 64, False), (56, 1280, 64, False), (72, 1100, 64, False),
    (300, 300, 64, False), (160, 1024, 64, False), (1024, 100, 64, False),
])
def test_equals_separate_passes(H, S, D, causal):
    from tests import gpu_util as G

    cfg, bits = I.random_case_bits(7300 + S + H, 1, H, S, D)
    one = G.run_fwd_bwd(bits, cfg.scale, causal)
    two = G.run_fwd_bwd(bits, cfg.scale, causal, fused_bwd=False)
    for n in ("dq", "dk", "dv"):
        assert bool(one[n].isfinite().all()), n
        assert torch.equal(one[n], two[n]), n
    heads = sorted({0, H // 2, H - 1})
    x = {t: I.bf16_bits_to_float(bits[t][:, heads]) for t in bits}
    ref = A.attn_bwd_ref(x["q"], x["k"], x["v"], x["dO"], cfg.scale, causal)
    for n in ("dq", "dk", "dv"):
        G.check(n, G.to_f64(one[n][:, heads].contiguous()), ref[n])
