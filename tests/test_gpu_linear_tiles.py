"""The linear layer where its tile kinds meet their edges: token counts one short of, at and one past a tile, a second
128-column half that is missing, one or two stages of contraction, and token ranges of uneven length in dw."""
import numpy as np
import pytest
import torch

from oracle import linear_ref as L
from paper_2507_00394_amd import inputs as I
from tests.dispatch_host import ask
from tests.test_gpu_parity_linear import _check_bf16, _check_f32

pytestmark = pytest.mark.gpu


# edge of the tile; the last: a missing column half
@pytest.mark.parametrize("edge,M,K,N", [(64, 1, 128, 128), (64, 63, 128, 384), (64, 65, 256, 128), (64, 129, 2048, 768), (128, 8191, 256, 384), (128, 8193, 1024, 768),
                                        (128, 32769, 128, 2688), (256, 16129, 2048, 896)])
def test_forward_edges(edge, M, K, N):
    assert ask([(M, K, N)], "tile_edge(linear_tile(M, K, N))", names=("M", "K", "N")) == [(edge,)]
    from paper_2507_00394_amd import binding as hx
    from tests import gpu_util as G

    bits = I.linear_case_bits(31 + M + K + N, M, K, N)
    guard = torch.full((M + 1, N), float("nan"), dtype=torch.bfloat16, device="cuda")
    hx.helix_qkv_linear_fwd(G.to_dev(bits["a"]), G.to_dev(bits["w"]), guard[:M])
    torch.cuda.synchronize()
    _check_bf16("qkv", G.to_f64(guard[:M]), L.linear_fwd_ref(I.bf16_bits_to_float(bits["a"]), I.bf16_bits_to_float(bits["w"])))
    assert torch.isnan(guard[M]).all()


# edges of the tiles of da and dw; dw over up to seven token ranges of uneven length
@pytest.mark.parametrize("input,weight,M,K,N", [(64, 64, 32, 128, 384), (64, 64, 96, 384, 128), (128, 128, 2080, 2048, 768), (128, 128, 16352, 640, 1408),
                                                (128, 128, 6176, 384, 2304), (128, 64, 4128, 128, 640), (256, 256, 8160, 1920, 2048)])
def test_backward_edges(input, weight, M, K, N):
    edges = [f"tile_edge(linear_gradient_tiles(M, K, N, linear_bwd_weight_parts(M, K, N)).{x})" for x in ("input", "weight")]
    assert ask([(M, K, N)], *edges, names=("M", "K", "N")) == [(input, weight)]
    from paper_2507_00394_amd import binding as hx
    from tests import gpu_util as G

    bits = I.linear_case_bits(57 + M + K + N, M, K, N)
    da = torch.full((M, K), float("nan"), dtype=torch.bfloat16, device="cuda")
    dw = torch.full((K, N), float("nan"), dtype=torch.float32, device="cuda")
    ws = torch.empty(hx.helix_qkv_linear_bwd_workspace_bytes(M, K, N), dtype=torch.uint8, device="cuda")
    hx.helix_qkv_linear_bwd(G.to_dev(bits["a"]), G.to_dev(bits["w"]), G.to_dev(bits["dqkv"]), da, dw, ws)
    torch.cuda.synchronize()
    f = {t: I.bf16_bits_to_float(bits[t]) for t in bits}
    ref = L.linear_bwd_ref(f["a"], f["w"], f["dqkv"])
    _check_bf16("da", G.to_f64(da), ref["da"])
    _check_f32("dw", G.to_f64(dw), ref["dw"])
