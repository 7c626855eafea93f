"""NaN and infinity in the inputs of the forward.  A NaN score reaches O and LSE of every row that sees it, wherever in the row it
stands: also where it is all that one of the two or four key groups of a workgroup holds for that row (a maximum does not see it).
A score of -inf takes its key out.  Rows that see neither are as without them.  Few heads and many, both masks."""
import numpy as np
import pytest
import torch

from oracle import attention_ref as A
from paper_2507_00394_amd import inputs as I
from tests.dispatch_host import ask

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


def _four_groups(S, causal):
    """Two heads of S tokens at head dimension 128 take the kernel with four key groups: group g has keys 32 g .. 32 g + 31 of every 128."""
    assert ask([(128, 2, S, causal)], "forward_rows(D, BH, S, causal)") == [(3,)]


# the first key of a group, all that a row has of it; a whole block; one block of a later tile, and the last, ragged one
@pytest.mark.parametrize("causal", [True, False])
@pytest.mark.parametrize("S,bad", [(673, (32, 33)), (673, (64, 65)), (673, (96, 97)), (673, (64, 96)), (673, (96, 128)), (673, (0, 1)), (673, (544, 545)), (673, (672, 673)),
                                   (1500, (32, 64)), (1500, (1376, 1377)), (1500, (1472, 1500))])
def test_nan_keys_in_four_groups(S, bad, causal):
    _four_groups(S, causal)
    test_nan_keys_reach_every_row_that_sees_them(S, bad, causal, 128, 2)


def test_nan_query_row_in_four_groups():
    _four_groups(673, True)
    test_nan_query_row(673, 128, True, 2)


# every key of a group goes; of the first group, as in the kernels without groups, all but the first block
@pytest.mark.parametrize("causal", [True, False])
@pytest.mark.parametrize("group", [0, 1, 2, 3])
def test_scores_of_minus_infinity_in_one_of_four_groups(group, causal):
    from tests import gpu_util as G

    S, D = 673, 128
    _four_groups(S, causal)
    x = _inputs(S, D)
    x["q"][:, 0] = 1.0
    gone = (np.arange(S) // 32) % 4 == group
    if group == 0:
        gone[:32] = False
    x["k"][gone, 0] = -np.inf
    o, lse = _forward(x, causal, D ** -0.5, 2)
    s = x["q"] @ np.where(gone[:, None], 0.0, x["k"]).T * D ** -0.5
    s[:, gone] = -np.inf
    if causal:
        s[np.triu_indices(S, 1)] = -np.inf
    m = s.max(1, keepdims=True)
    p = np.exp(s - m)
    G.check("o", o, p / p.sum(1, keepdims=True) @ x["v"])
    assert np.abs(lse - (m[:, 0] + np.log(p.sum(1)))).max() <= G.TOL_LSE
