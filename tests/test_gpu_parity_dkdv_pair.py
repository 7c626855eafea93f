"""The head-dimension-128 dK/dV pass walks a key tile's query blocks in regimes: pipelined steps
with a general copy in front for the first blocks (one; with a causal mask the four that the
diagonal cuts), groups of seven blocks with the copies inside the steps, the first kind of step
again for the complete blocks that are left, and a plain path for a ragged last block.  The sequence lengths here put the boundaries between the regimes at every
remainder of the seven-block groups, with whole and ragged last blocks, for full and causal
attention; every result is compared with the fp64 oracle element by element.  Two heads take key tiles of 64 keys and two pairs of
waves, more of them 128 keys and four pairs; a test asserts which."""
import pytest

from oracle import attention_ref as A
from paper_2507_00394_amd import inputs as I
from tests.dispatch_host import ask

pytestmark = pytest.mark.gpu

# full attention: every key tile sees S // 32 whole blocks; the first group of seven needs 14 of them
# (one before it, and what its copies ahead may touch)
FULL = [32 * 13, 32 * 14, 32 * 14 + 1, 32 * 15 + 31, 32 * 16, 32 * 17 + 5, 32 * 18, 32 * 19 + 30, 32 * 20, 32 * 21 + 1,
        32 * 22, 32 * 28 + 17, 32 * 35]
# causal: key tile t sees (S - 128 t) // 32 blocks, so one length covers many remainders at once
CAUSAL = [32 * 20, 32 * 21 + 9, 1216, 1409, 2047, 2304]


def _check(S, causal, seed):
    from tests import gpu_util as G

    cfg, bits = I.random_case_bits(seed, 1, 2, S, 128)
    out = G.run_fwd_bwd(bits, cfg.scale, causal)
    f = {t: I.bf16_bits_to_float(bits[t]) for t in bits}
    ref = A.attn_bwd_ref(f["q"], f["k"], f["v"], f["dO"], cfg.scale, causal)
    for n in ("dk", "dv", "dq", "o"):
        G.check(n, G.to_f64(out[n]), ref[n])


def _key_tile(H, S, causal):
    return ask([(128, H, S, causal)], "key_tile(gradient_tiles(D, BH, S, causal))")[0][0]


@pytest.mark.parametrize("S", FULL)
def test_full_attention_block_regimes(S):
    assert _key_tile(2, S, False) == 64
    _check(S, False, 7100 + S)


@pytest.mark.parametrize("S", CAUSAL)
def test_causal_block_regimes(S):
    assert _key_tile(2, S, True) == 64
    _check(S, True, 7200 + S)


# as many heads as it takes for 128-key tiles; the shortest sweeps too: no, one and few whole blocks, and the diagonal's four
@pytest.mark.parametrize("H,S,causal", [(72, 95, False), (38, 225, False)] + [(24, s, False) for s in FULL[:6]] + [(17, s, False) for s in FULL[6:]] +
                         [(76, 96, True), (76, 127, True), (76, 128, True), (60, 129, True), (60, 161, True), (48, 255, True), (32, 512, True), (30, 547, True), (30, 576, True)] +
                         [(26, s, True) for s in CAUSAL])
def test_wide_key_tiles(H, S, causal):
    from tests import gpu_util as G

    assert _key_tile(H, S, causal) == 128
    cfg, bits = I.random_case_bits(7400 + S, 1, H, S, 128)
    out = G.run_fwd_bwd(bits, cfg.scale, causal)
    heads = [0, H - 1]
    f = {t: I.bf16_bits_to_float(bits[t][:, heads]) for t in bits}
    ref = A.attn_bwd_ref(f["q"], f["k"], f["v"], f["dO"], cfg.scale, causal)
    for n in ("dk", "dv"):
        assert bool(out[n].isfinite().all()), n
        G.check(n, G.to_f64(out[n][:, heads].contiguous()), ref[n])


def test_full_attention_many_groups_and_ragged_end():
    """Full attention at a length with 36 seven-block groups per key tile and a ragged last block: every key tile
    runs groups of seven from its second block on (there is no diagonal) for hundreds of blocks."""
    _check(32 * 259 + 17, False, 7300)
