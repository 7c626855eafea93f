"""The delta of the first rows on grids that fill the chip with 256-row or (head dimension 128) 128-row tiles: the same bits as for a few of the heads
alone, whose small grid takes 64-row tiles (held against the oracle elsewhere).  Lengths at the edges of a wave's 32 rows, of the 64-key tiles and of
the row tiles, and more rows than delta_head covers."""
import pytest
import torch

from paper_2507_00394_amd import inputs as I
from tests.dispatch_host import ask

pytestmark = pytest.mark.gpu

K256, K128, K64 = 0, 1, 2


@pytest.mark.parametrize("kind,H,S,D,causal", [
    (K256, 203, 191, 64, True), (K256, 217, 600, 64, True), (K256, 62, 2049, 64, True), (K256, 58, 2304, 64, True),
    (K256, 385, 250, 64, False), (K256, 209, 257, 64, False), (K256, 167, 513, 64, False), (K256, 49, 2049, 64, False),
    (K256, 409, 250, 128, True), (K256, 187, 600, 128, True), (K256, 75, 1537, 128, True), (K256, 60, 2049, 128, True),
    (K256, 385, 250, 128, False), (K256, 373, 257, 128, False), (K256, 191, 513, 128, False), (K256, 51, 2304, 128, False),
    (K128, 414, 65, 128, True), (K128, 107, 129, 128, True), (K128, 121, 250, 128, True), (K128, 174, 257, 128, True), (K128, 71, 600, 128, True),
    (K128, 34, 1537, 128, True), (K128, 28, 2049, 128, True),
    (K128, 414, 65, 128, False), (K128, 135, 257, 128, False), (K128, 86, 600, 128, False), (K128, 36, 2304, 128, False)])
def test_same_bits_as_small_grid(kind, H, S, D, causal):
    from paper_2507_00394_amd import binding as hx
    from tests import gpu_util as G

    rows = min(S, hx.DELTA_HEAD_ROWS)
    some = [0, H // 2, H - 1]
    assert [k for k, in ask([(D, H, rows, causal), (D, len(some), rows, causal)], "delta_rows(D, BH, S, causal)")] == [kind, K64]
    cfg, bits = I.random_case_bits(9900 + S + H, 1, H, S, D)
    planes = []
    for heads in (list(range(H)), some):
        q, k, v, g = (G.to_dev(bits[t][:, heads].copy()) for t in ("q", "k", "v", "dO"))
        o, lse = torch.empty_like(q), torch.empty(1, len(heads), S, dtype=torch.float32, device="cuda")
        hx.helix_attn_fwd(q, k, v, o, lse, cfg.scale, causal)
        if len(planes) == 0:
            lse_all = lse
        else:
            lse = lse_all[:, some].contiguous()   # the forward's bits may depend on the grid
        stats = torch.full((hx.helix_attn_bwd_workspace_bytes(1, len(heads), S, D),), 0xff, dtype=torch.uint8, device="cuda")
        hx.helix_attn_bwd_delta_head(q, k, v, g, lse, stats, hx.DELTA_HEAD_ROWS, cfg.scale, causal)
        torch.cuda.synchronize()
        planes.append(stats[:len(heads) * S * 4].view(torch.float32).reshape(len(heads), S)[:, :rows].clone())
    assert bool(planes[0].isfinite().all())
    assert torch.equal(planes[0][some], planes[1])
