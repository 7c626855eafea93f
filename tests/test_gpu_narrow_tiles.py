"""Narrow workgroups (64 rows or keys, four waves), which small grids take in every pass: lengths at the edges of their 32-row groups, of
the 64-key tiles and of the query halves, a few grids that take the wider ones in some passes, and the same bits as the 128-row workgroups."""
import numpy as np
import pytest
import torch

from oracle import attention_ref as A
from paper_2507_00394_amd import inputs as I
from tests.dispatch_host import ask

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("causal", [True, False])
@pytest.mark.parametrize("H,S", [(1, 1), (2, 31), (5, 33), (1, 63), (3, 95), (2, 127), (7, 129), (2, 191), (4, 193), (9, 257), (1, 700), (3, 1000),
                                 (7, 1300), (9, 2100), (60, 333), (40, 1100)])
def test_edges(H, S, causal, D):
    from tests import gpu_util as G

    cfg, bits = I.random_case_bits(6200 + S + H, 1, H, S, D)
    out = G.run_fwd_bwd(bits, cfg.scale, causal)
    for n in ("o", "lse", "dq", "dk", "dv"):
        assert bool(torch.isfinite(out[n].float()).all()), n
    heads = sorted({0, H // 2, H - 1})
    x = {t: I.bf16_bits_to_float(bits[t][:, heads]) for t in bits}
    ref = A.attn_bwd_ref(x["q"], x["k"], x["v"], x["dO"], cfg.scale, causal)
    for n in ("o", "dq", "dk", "dv"):
        G.check(n, G.to_f64(out[n][:, heads].contiguous()), ref[n])
    assert np.abs(G.to_f64(out["lse"][:, heads]) - ref["lse"]).max() <= G.TOL_LSE


# Keys in four groups (head dimension 128, few heads, no short sequence): tokens at the edges of the 32-key blocks of a 128-key tile and of the
# 64-row tiles, rows that see one, two, three and all of the groups of their last tile
@pytest.mark.parametrize("causal", [True, False])
@pytest.mark.parametrize("H,S", [(2, 640), (1, 641), (3, 671), (2, 672), (1, 673), (2, 703), (1, 736), (3, 737), (2, 767), (1, 769), (5, 1500), (2, 2113)])
def test_four_key_groups(H, S, causal):
    assert ask([(128, H, S, causal)], "forward_rows(D, BH, S, causal)") == [(3,)]
    test_edges(H, S, causal, 128)


@pytest.mark.parametrize("causal", [True, False])
def test_four_key_groups_on_views(causal):
    """Views of a fused [S, B, 3, H, D] buffer, read and written by four key groups: the bits of contiguous tensors."""
    from paper_2507_00394_amd import binding as hx
    from tests import gpu_util as G

    B, H, S, D = 2, 2, 717, 128
    assert ask([(D, B * H, S, causal)], "forward_rows(D, BH, S, causal)") == [(3,)]
    cfg, bits = I.random_case_bits(6500, B, H, S, D)
    whole = G.run_fwd_bwd(bits, cfg.scale, causal)
    qkv = torch.full((S, B, 3, H, D), float("nan"), dtype=torch.bfloat16, device="cuda")
    q, k, v = (qkv[:, :, i].permute(1, 2, 0, 3) for i in range(3))
    for view, t in ((q, "q"), (k, "k"), (v, "v")):
        view.copy_(whole[t])
    o = torch.full((S, B, H, D + 8), float("nan"), dtype=torch.bfloat16, device="cuda")
    lse = torch.full((B, H, S), float("nan"), device="cuda")
    hx.helix_attn_fwd_strided(q, k, v, o[..., :D].permute(1, 2, 0, 3), lse, cfg.scale, causal)
    torch.cuda.synchronize()
    assert torch.equal(o[..., :D].permute(1, 2, 0, 3), whole["o"]) and torch.equal(lse, whole["lse"])
    assert bool(o[..., D:].isnan().all())


# Many heads against two of them alone, which take narrow workgroups: the forward at head dimension 64, and the gradients from the same O and LSE.  (At head
# dimension 64 a causal key tile's rows are halved from its first key on, so dK and dV of narrow tiles are sums in another order.)
FORWARD, GRADIENTS = "forward_rows(D, BH, S, causal)", "gradient_tiles(D, BH, S, causal)"
K128, K64, TOGETHER_128, NARROW = 1, 2, 3, 4


@pytest.mark.parametrize("H,S,D,causal,rule,many_kind,few_kind,same", [
    (24, 1500, 128, True, GRADIENTS, TOGETHER_128, NARROW, ("dq", "dk", "dv")), (30, 777, 128, False, GRADIENTS, TOGETHER_128, NARROW, ("dq", "dk", "dv")),
    (130, 257, 64, True, GRADIENTS, TOGETHER_128, NARROW, ("dq",)), (40, 700, 64, False, GRADIENTS, TOGETHER_128, NARROW, ("dq", "dk", "dv")),
    (200, 333, 64, True, FORWARD, K128, K64, ("o", "lse")), (200, 333, 64, False, FORWARD, K128, K64, ("o", "lse"))])
def test_bits_of_a_head_alone(H, S, D, causal, rule, many_kind, few_kind, same):
    from paper_2507_00394_amd import binding as hx
    from tests import gpu_util as G

    assert ask([(D, H, S, causal), (D, 2, S, causal)], rule) == [(many_kind,), (few_kind,)]
    cfg, bits = I.random_case_bits(6300 + S, 1, H, S, D)
    many = G.run_fwd_bwd(bits, cfg.scale, causal)
    few = {n: many[n][:, H - 2:].contiguous() for n in ("q", "k", "v", "dO")}
    few.update({n: torch.full_like(few["q"], float("nan")) for n in ("o", "dq", "dk", "dv")}, lse=torch.full((1, 2, S), float("nan"), device="cuda"))
    hx.helix_attn_fwd(few["q"], few["k"], few["v"], few["o"], few["lse"], cfg.scale, causal)
    ws = torch.empty(hx.helix_attn_bwd_workspace_bytes(1, 2, S, D), dtype=torch.uint8, device="cuda")
    o, lse = many["o"][:, H - 2:].contiguous(), many["lse"][:, H - 2:].contiguous()
    hx.helix_attn_bwd(few["q"], few["k"], few["v"], o, lse, few["dO"], few["dq"], few["dk"], few["dv"], ws, cfg.scale, causal)
    torch.cuda.synchronize()
    for n in same:
        assert torch.equal(many[n][:, H - 2:], few[n]), n


def test_stage_calls_take_the_same_tiles():
    """The backward's stages one by one are the whole backward bit for bit."""
    from tests import gpu_util as G

    for H, S, D, causal in ((3, 500, 128, True), (3, 500, 64, True), (2, 333, 64, False), (2, 333, 128, False)):
        cfg, bits = I.random_case_bits(6400 + S, 1, H, S, D)
        a, b = G.run_fwd_bwd(bits, cfg.scale, causal), G.run_fwd_bwd(bits, cfg.scale, causal, fused_bwd=False)
        for n in ("dq", "dk", "dv"):
            assert torch.equal(a[n], b[n]), (n, H, S, D, causal)
