"""zc_dequantize_cache of ROW layout around the size from which a thread expands four slots, and above it: ragged
last quads, every bit width, token scales and none, exactly the unpacked cache in token order."""
import pytest
import torch

from paper_2405_14256_amd import binding as zb
from tests.test_gpu_literal import _unpacked

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("L", [4095, 4096, 4099, 4102])          # 2^20 vectors at 4096 tokens
@pytest.mark.parametrize("bits_hi,bits_lo,k,scheme,dtype", [(4, 2, 1633, "channel", torch.bfloat16), (8, 4, 1, "channel", torch.float16),
                                                            (2, 8, 0, "token", torch.float32)])
def test_dequantize_row_quads(L, bits_hi, bits_lo, k, scheme, dtype):
    B, H, d = 2, 8, 128
    g = torch.Generator().manual_seed(L)
    x = torch.randn(B, H, L, d, generator=g).to(dtype).to("cuda")
    p = zb.PackedTensor(B, H, d, 1664, 4160, bits_hi, bits_lo, scheme, zb.ZC_LAYOUT_ROW, max_chunks=1, device="cuda")
    sal, reg = zb.zc_select_salient(torch.rand(B, L, generator=g).cuda(), k)
    zb.zc_quantize_pack(x, sal, reg, p)
    out = torch.zeros_like(x)
    zb.zc_dequantize_cache(p, out)
    assert torch.equal(out, _unpacked(p, L, dtype))


@pytest.mark.parametrize("L", [2047, 2048, 2051])                 # 2^19 vectors at 2048 tokens
@pytest.mark.parametrize("bits_hi,bits_lo,k,scheme,dtype", [(4, 2, 821, "channel", torch.float16), (8, 4, 1023, "token", torch.bfloat16)])
def test_dequantize_row_quads_from_half_that_size(L, bits_hi, bits_lo, k, scheme, dtype):
    test_dequantize_row_quads(L, bits_hi, bits_lo, k, scheme, dtype)


@pytest.mark.parametrize("L", [2559, 2560, 2563])                 # 5 * 2^18 vectors at 2560 tokens, where fp32 starts
@pytest.mark.parametrize("bits_hi,bits_lo,k,scheme", [(4, 2, 1025, "channel"), (8, 4, 5, "token")])
def test_dequantize_row_quads_of_fp32(L, bits_hi, bits_lo, k, scheme):
    B, H, d = 4, 8, 128
    g = torch.Generator().manual_seed(L)
    x = torch.randn(B, H, L, d, generator=g).to("cuda")
    p = zb.PackedTensor(B, H, d, 1088, 2624, bits_hi, bits_lo, scheme, zb.ZC_LAYOUT_ROW, max_chunks=1, device="cuda")
    sal, reg = zb.zc_select_salient(torch.rand(B, L, generator=g).cuda(), k)
    zb.zc_quantize_pack(x, sal, reg, p)
    out = torch.zeros_like(x)
    zb.zc_dequantize_cache(p, out)
    assert torch.equal(out, _unpacked(p, L, torch.float32))
