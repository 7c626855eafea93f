"""What a head's results depend on beside the head: its batch and its neighbours decide, through the size of the grid, which tiles a pass
takes, and with them the order of its sums.  One call with several samples against a call per sample, at sizes where the two lie on
different sides of a rule.  A rounding to bf16 is within 2^-8.  O: P is rounded against another reference maximum, so either result is within
2^-8 sum_j p_ij |v_jd| of the exact one before it is itself rounded.  Gradients from the same O and LSE: the same dS and P in bf16, only the
order of the fp32 sums differs, by far less than 1e-4 of their root mean square, and the two results are rounded once each."""
import numpy as np
import pytest
import torch

from paper_2507_00394_amd import inputs as I

pytestmark = pytest.mark.gpu


def _within(a, b, extra):
    a, b = a.double(), b.double()
    return bool(((a - b).abs() <= 2.0 ** -7 * torch.maximum(a.abs(), b.abs()) + extra).all())


# B, H, S, D, causal; the outputs that are the same bits whatever else is in the call, and one at least that is not
@pytest.mark.parametrize("B,H,S,D,causal,same,differs", [
    (2, 32, 2048, 128, True, ("dk", "dv"), "o"),
    (4, 8, 1500, 128, False, ("dk", "dv"), "o"),
    (8, 12, 1024, 64, True, ("o", "lse"), "dk"),
    (8, 8, 1024, 64, False, ("o", "lse"), "dk"),
])
def test_samples_together_and_alone(B, H, S, D, causal, same, differs):
    from paper_2507_00394_amd import binding as hx
    from tests import gpu_util as G

    cfg, bits = I.random_case_bits(3300 + S, B, H, S, D)
    x = {t: G.to_dev(bits[t]) for t in bits}

    def run(t, o=None, lse=None):
        out = {n: torch.full_like(t["q"], float("nan")) for n in ("o", "dq", "dk", "dv")}
        out["lse"] = torch.full(t["q"].shape[:3], float("nan"), dtype=torch.float32, device="cuda")
        hx.helix_attn_fwd(t["q"], t["k"], t["v"], out["o"], out["lse"], cfg.scale, causal)
        ws = torch.empty(hx.helix_attn_bwd_workspace_bytes(*t["q"].shape), dtype=torch.uint8, device="cuda")
        hx.helix_attn_bwd(t["q"], t["k"], t["v"], out["o"] if o is None else o, out["lse"] if lse is None else lse, t["dO"], out["dq"], out["dk"],
                          out["dv"], ws, cfg.scale, causal)
        return out

    both = run(x)
    for b in (0, B - 1):
        t = {n: v[b:b + 1].contiguous() for n, v in x.items()}
        one = run(t, both["o"][b:b + 1].contiguous(), both["lse"][b:b + 1].contiguous())
        weight = torch.empty_like(t["q"])   # sum_j p_ij |v_jd|
        hx.helix_attn_fwd(t["q"], t["k"], t["v"].abs(), weight, torch.empty_like(one["lse"]), cfg.scale, causal)
        torch.cuda.synchronize()
        for n in ("o", "lse", "dq", "dk", "dv"):
            p, q = both[n][b], one[n][0]
            assert bool(p.isfinite().all()) and bool(q.isfinite().all()), n
            if n in same:
                assert torch.equal(p, q), n
            elif n == "lse":
                assert (p - q).abs().max().item() <= 1e-5
            else:
                extra = 2.0 ** -7 * 1.01 * weight[0].double() if n == "o" else 1e-4 * q.double().square().mean().sqrt()
                assert _within(p, q, extra), n
        assert not torch.equal(both[differs][b], one[differs][0])   # else the case does not straddle a rule
