"""The delta of the first rows on grids that fill the chip with 256-row tiles: the same bits as for a few of the heads alone,
whose small grid takes 128-row tiles with the key halves in two groups of waves (held against the oracle elsewhere).  Lengths at the
edges of a wave's 32 rows, of the 64-key tiles and of both row tiles, and more rows than delta_head covers."""
import pytest
import torch

from paper_2507_00394_amd import inputs as I

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("H,S,D", [(257, 1, 64), (257, 33, 128), (260, 65, 64), (260, 256, 128), (130, 257, 128), (100, 600, 64), (43, 1537, 128),
                                   (33, 2049, 128), (33, 2304, 64),
                                   (192, 256, 128), (128, 257, 128), (96, 600, 64), (48, 1537, 128), (40, 2049, 128), (40, 2304, 64)])
@pytest.mark.parametrize("causal", [True, False])
def test_same_bits_as_small_grid(H, S, D, causal):
    from paper_2507_00394_amd import binding as hx
    from tests import gpu_util as G

    cfg, bits = I.random_case_bits(9900 + S + H, 1, H, S, D)
    some = [0, H // 2, H - 1]
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
        rows = min(S, hx.DELTA_HEAD_ROWS)
        planes.append(stats[:len(heads) * S * 4].view(torch.float32).reshape(len(heads), S)[:, :rows].clone())
    assert bool(planes[0].isfinite().all())
    assert torch.equal(planes[0][some], planes[1])
