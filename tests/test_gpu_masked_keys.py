"""Delta of the first rows: a key block that lies wholly above the causal diagonal of a wave's rows is not touched, whatever V holds
there, on grids of 64-row, 128-row and 256-row tiles."""
import pytest
import torch

from paper_2507_00394_amd import inputs as I
from tests.dispatch_host import ask

pytestmark = pytest.mark.gpu


K256, K128, K64 = 0, 1, 2


@pytest.mark.parametrize("kind,H,S,D", [(K64, 3, 64, 64), (K64, 3, 200, 128), (K64, 300, 64, 64), (K64, 300, 64, 128), (K128, 300, 200, 128), (K256, 192, 200, 128),
                                        (K256, 203, 191, 64)])
def test_delta_of_rows_that_do_not_see_an_infinite_value(kind, H, S, D):
    assert ask([(D, H, S, True)], "delta_rows(D, BH, S, causal)") == [(kind,)]
    from paper_2507_00394_amd import binding as hx
    from tests import gpu_util as G

    cfg, bits = I.random_case_bits(6200 + S, 1, H, S, D)
    q, k, v, g = (G.to_dev(bits[t]) for t in ("q", "k", "v", "dO"))
    o, lse = torch.empty_like(q), torch.empty(1, H, S, dtype=torch.float32, device="cuda")
    hx.helix_attn_fwd(q, k, v, o, lse, cfg.scale, True)
    planes = []
    for value in (None, float("inf"), float("nan")):
        if value is not None:
            v[:, :, 40] = value
        stats = torch.full((hx.helix_attn_bwd_workspace_bytes(1, H, S, D),), 0xff, dtype=torch.uint8, device="cuda")
        hx.helix_attn_bwd_delta_head(q, k, v, g, lse, stats, hx.DELTA_HEAD_ROWS, cfg.scale, True)
        torch.cuda.synchronize()
        planes.append(stats[:H * S * 4].view(torch.float32).reshape(H, S).clone())
    for p in planes[1:]:
        assert torch.equal(p[:, :32], planes[0][:, :32])   # the wave's rows 0..31 see keys 0..31 only
        assert not p[:, 40:].isfinite().any()
