"""Decode over caches with 8-bit codes: blocks of 16 slots, a code at its exact fp16 value."""
import pytest
import torch

from paper_2405_14256_amd import binding as zb

pytestmark = pytest.mark.gpu
DEV = "cuda"


@pytest.mark.parametrize("bits", [(8, 8), (8, 4), (8, 2), (2, 8), (4, 8)])
@pytest.mark.parametrize("dtype,d,B,Hkv,G", [(torch.float32, 128, 1, 2, 4), (torch.float32, 64, 2, 1, 8), (torch.bfloat16, 128, 2, 3, 1),
                                             (torch.float16, 64, 70, 4, 2), (torch.float16, 128, 64, 5, 4)])
def test_decode_with_8_bit_codes(bits, dtype, d, B, Hkv, G):
    """Segments that end at, before and after a block's edge, empty subsets, every scheme on
    either tensor, launches below and above one workgroup per compute unit, against attention
    in float64 over the de-quantized cache."""
    g = torch.Generator().manual_seed(d * B + bits[0])
    lib = zb.load()
    sizes = [(33, 47), (16, 15), (0, 17), (1, 0), (64, 64)]
    T = 19
    n = sum(a + b for a, b in sizes)
    X = torch.randn(2, B, Hkv, n + T, d, generator=g).to(dtype).to(DEV)
    q = torch.randn(B, Hkv * G, d, generator=g).to(dtype).to(DEV)
    for k_scheme, v_scheme in (("channel", "cst"), ("token", "channel"), ("cst", "token")):
        mk = lambda s, layout: zb.PackedTensor(B, Hkv, d, lib.zc_arena_slots(114, 5), lib.zc_arena_slots(143, 5), *bits, s, layout,
                                               max_chunks=5, device=DEV)
        Kp, Vp = mk(k_scheme, zb.ZC_LAYOUT_ROW), mk(v_scheme, zb.ZC_LAYOUT_TGROUP)
        at = 0
        for k, r in sizes:
            sal, reg = zb.zc_select_salient(torch.rand(B, k + r, generator=g).to(DEV), k)
            for x, p in ((X[0], Kp), (X[1], Vp)):
                zb.zc_quantize_pack(x[:, :, at:at + k + r], sal, reg, p, pos_offset=at)
            at += k + r
        Kh, Vh = X[0].float(), X[1].float()
        zb.zc_dequantize_cache(Kp, Kh)
        zb.zc_dequantize_cache(Vp, Vh)
        lse = torch.empty(B, Hkv * G, dtype=torch.float32, device=DEV)
        out = zb.zc_decode_attention(q, Kp, Vp, X[0][:, :, n:], X[1][:, :, n:], T, lse_out=lse)
        logits = (q.double().view(B, Hkv, G, 1, d) * Kh.double()[:, :, None]).sum(-1).view(B, Hkv * G, -1) / d ** 0.5
        want_lse = torch.logsumexp(logits, -1)
        p = torch.exp(logits - want_lse[..., None]).view(B, Hkv, G, -1, 1)
        want = (p * Vh.double()[:, :, None]).sum(-2).view(B, Hkv * G, d)
        # fp32: sums of d and n terms below 10 in fp32, query and weights to 22 bits; 16-bit tensors:
        # the weights' and the output's rounding
        tol = {torch.float32: 1e-5, torch.float16: 2e-3, torch.bfloat16: 1.6e-2}[dtype]
        assert float((out.double() - want).abs().max()) <= tol, (k_scheme, v_scheme)
        assert float((lse.double() - want_lse).abs().max()) <= min(tol, 1e-3), (k_scheme, v_scheme)
