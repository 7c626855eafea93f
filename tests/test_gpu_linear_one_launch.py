"""The linear layer's two gradients, in their common launch or one each: shapes for the pairs of tiles, with workgroup
counts that are no multiple of the XCDs, ragged token tiles and, in the last ones, a weight gradient in parts."""
import pytest
import torch

from oracle import linear_ref as L
from paper_2507_00394_amd import inputs as I
from tests.dispatch_host import ask
from tests.test_gpu_parity_linear import _check_bf16, _check_f32

pytestmark = pytest.mark.gpu


# edges of the input and of the weight gradient's tile; whether the weight gradient comes in parts
@pytest.mark.parametrize("input,weight,in_parts,M,K,N", [
    (64, 64, False, 32, 384, 128), (64, 64, True, 4128, 128, 1152), (64, 128, False, 224, 1280, 1280), (64, 128, True, 6176, 256, 1408), (128, 64, False, 608, 256, 128),
    (128, 64, True, 6176, 256, 384), (128, 128, False, 608, 4992, 256), (128, 128, True, 4128, 2048, 256), (256, 256, False, 1504, 4096, 1792),
    (256, 256, True, 6176, 1280, 1536), (64, 256, False, 32, 12544, 2048), (128, 256, False, 224, 12032, 1792), (128, 256, True, 65568, 384, 896)])
def test_gradients_in_one_launch(input, weight, in_parts, M, K, N):
    edges = [f"tile_edge(linear_gradient_tiles(M, K, N, linear_bwd_weight_parts(M, K, N)).{x})" for x in ("input", "weight")]
    assert ask([(M, K, N)], *edges, "linear_bwd_weight_parts(M, K, N) > 1", names=("M", "K", "N")) == [(input, weight, in_parts)]
    from paper_2507_00394_amd import binding as hx
    from tests import gpu_util as G

    bits = I.linear_case_bits(71 + M + K + N, M, K, N)
    da = torch.full((M + 1, K), float("nan"), dtype=torch.bfloat16, device="cuda")
    dw = torch.full((K + 1, N), float("nan"), dtype=torch.float32, device="cuda")
    ws = torch.empty(hx.helix_qkv_linear_bwd_workspace_bytes(M, K, N), dtype=torch.uint8, device="cuda")
    hx.helix_qkv_linear_bwd(G.to_dev(bits["a"]), G.to_dev(bits["w"]), G.to_dev(bits["dqkv"]), da[:M], dw[:K], ws)
    torch.cuda.synchronize()
    f = {t: I.bf16_bits_to_float(bits[t]) for t in bits}
    ref = L.linear_bwd_ref(f["a"], f["w"], f["dqkv"])
    _check_bf16("da", G.to_f64(da[:M]), ref["da"])
    _check_f32("dw", G.to_f64(dw[:K]), ref["dw"])
    assert torch.isnan(da[M]).all() and torch.isnan(dw[K]).all()
