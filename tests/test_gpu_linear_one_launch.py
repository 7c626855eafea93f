"""The linear layer's two gradients, in their common launch or one each: shapes for the pairs of tiles, with workgroup
counts that are no multiple of the XCDs, ragged token tiles and, in the last ones, a weight gradient in parts."""
import pytest
import torch

from oracle import linear_ref as L
from paper_2507_00394_amd import inputs as I
from tests.test_gpu_parity_linear import _check_bf16, _check_f32

pytestmark = pytest.mark.gpu


# input / weight tiles: 64 / 64, 128 / 64, 64 / 128, 128 / 128, 128 / 64 in parts, 256 / 256 in parts; one launch each: 64 / 256, 128 / 256, 256 / 128 in parts
@pytest.mark.parametrize("M,K,N", [(32, 384, 128), (224, 384, 128), (224, 1280, 1280), (608, 1152, 1152), (6176, 256, 384), (6176, 1280, 1536),
                                   (32, 12544, 2048), (224, 12032, 1792), (201024, 256, 640)])
def test_gradients_in_one_launch(M, K, N):
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
