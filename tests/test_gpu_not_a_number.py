"""NaN and infinity in the inputs of the forward.  A NaN score reaches O and LSE of every row that sees it, wherever in the row it
stands: also where it is all that one of the two key halves of a split workgroup holds for that row (a maximum does not see it).
A score of -inf takes its key out.  Rows that see neither are as without them.  Few heads and many, both masks."""
import numpy as np
import pytest
import torch

from oracle import attention_ref as A
from paper_2507_00394_amd import inputs as I

pytestmark = pytest.mark.gpu


def _forward(x, causal, scale, H):
    """x: q, k, v as float arrays [S, D] of one head; the same head H times."""
    from paper_2507_00394_amd import binding as hx

    q, k, v = (torch.from_numpy(x[t]).to(torch.bfloat16).cuda().expand(1, H, -1, -1).contiguous() for t in ("q", "k", "v"))
    o, lse = torch.zeros_like(q), torch.zeros(1, H, q.shape[2], dtype=torch.float32, device="cuda")
    hx.helix_attn_fwd(q, k, v, o, lse, scale, causal)
    torch.cuda.synchronize()
    assert torch.equal(o[0, 0].view(torch.int16), o[0, H - 1].view(torch.int16))
    return o[0, 0].double().cpu().numpy(), lse[0, 0].double().cpu().numpy()


def _inputs(S, D):
    _, bits = I.random_case_bits(640 + S, 1, 1, S, D)
    return {t: I.bf16_bits_to_float(bits[t])[0, 0] for t in ("q", "k", "v")}


@pytest.mark.parametrize("H", [2, 400])
@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("causal", [True, False])
@pytest.mark.parametrize("S,bad", [(33, (32, 33)), (64, (32, 33)), (64, (32, 64)), (80, (32, 33)), (80, (32, 64)), (96, (0, 32)), (200, (32, 64)),
                                   (200, (64, 96))])
def test_nan_keys_reach_every_row_that_sees_them(S, bad, causal, D, H):
    from tests import gpu_util as G

    x = _inputs(S, D)
    k = x["k"].copy()
    k[bad[0]:bad[1]] = np.nan
    o, lse = _forward(dict(x, k=k), causal, D ** -0.5, H)
    sees = np.arange(S) >= bad[0] if causal else np.ones(S, bool)
    assert np.isnan(o[sees]).all() and np.isnan(lse[sees]).all()
    if (~sees).any():
        ref, ref_lse = A.attn_fwd_ref(*(x[t][None, None, :bad[0]] for t in ("q", "k", "v")), D ** -0.5, causal)
        G.check("o", o[~sees], ref[0, 0])
        assert np.abs(lse[~sees] - ref_lse[0, 0]).max() <= G.TOL_LSE


@pytest.mark.parametrize("H", [2, 400])
@pytest.mark.parametrize("S,D,causal", [(33, 64, True), (64, 128, False), (80, 128, True), (200, 64, False)])
def test_nan_query_row(S, D, causal, H):
    x = _inputs(S, D)
    x["q"][5, 3] = np.nan
    o, lse = _forward(x, causal, D ** -0.5, H)
    row = np.arange(S) == 5
    assert np.isnan(o[row]).all() and np.isnan(lse[row]).all()
    assert np.isfinite(o[~row]).all() and np.isfinite(lse[~row]).all()


@pytest.mark.parametrize("H", [2, 400])
@pytest.mark.parametrize("S,D", [(64, 64), (64, 128), (96, 64), (96, 128)])
def test_score_of_minus_infinity_takes_its_key_out(S, D, H):
    from tests import gpu_util as G

    x = _inputs(S, D)
    x["q"][:, 0] = 1.0
    x["k"][32:64, 0] = -np.inf
    o, lse = _forward(x, False, D ** -0.5, H)
    keep = np.r_[0:32, 64:S]
    s = x["q"] @ x["k"][keep].T * D ** -0.5
    m = s.max(1, keepdims=True)
    p = np.exp(s - m)
    G.check("o", o, p / p.sum(1, keepdims=True) @ x["v"][keep])
    assert np.abs(lse - (m[:, 0] + np.log(p.sum(1)))).max() <= G.TOL_LSE
