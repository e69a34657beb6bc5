"""Prefill attention: the probe rows' normalisers, from the attention kernel itself and by a launch of their own."""
import pytest
import torch

from paper_2405_14256_amd import binding as zb

pytestmark = pytest.mark.gpu
DEV = "cuda"


# (dtype, d, B, Hq, Hkv, L, P): up to two probes a thread come from the kernel - workgroups of 512, 256, 128 and
# 64 threads (fp32, by heads and length), 256 and 512 (16 bit) - one more takes the other launch
@pytest.mark.parametrize("dtype,d,B,Hq,Hkv,L", [(torch.float32, 64, 1, 3, 1, 97), (torch.float32, 64, 2, 160, 160, 250),
                                                (torch.float32, 128, 1, 128, 32, 800), (torch.float32, 64, 2, 200, 200, 350),
                                                (torch.float16, 128, 2, 4, 2, 391),
                                                (torch.bfloat16, 64, 1, 8, 8, 33), (torch.bfloat16, 128, 1, 8, 1, 16400)])
@pytest.mark.parametrize("P", [1, 128, 129, 256, 257, 512, 513, 1024, 1025])
def test_probe_normalisers_are_the_rows(dtype, d, B, Hq, Hkv, L, P):
    """In any order, with repetitions; a position outside the prompt gets 0."""
    g = torch.Generator(device=DEV).manual_seed(P)
    q = torch.randn(B, Hq, L, d, generator=g, device=DEV).to(dtype)
    k, v = (torch.randn(B, Hkv, L, d, generator=g, device=DEV).to(dtype) for _ in range(2))
    pos = torch.randint(0, L, (P,), generator=g, device=DEV)
    pos[0], pos[-1] = L - 1, 0
    if P > 4:
        pos[2], pos[3] = L, -1
    lse_probe = torch.full((B, Hq, P), float("nan"), device=DEV)
    _, lse, got = zb.zc_prefill_attention(q, k, v, probe_pos=pos.int(), lse_probe=lse_probe)
    inside = (pos >= 0) & (pos < L)
    want = torch.where(inside, lse[:, :, pos.clamp(0, L - 1)], torch.zeros((), device=DEV))
    assert torch.equal(got, want)                       # moved, not computed: the same bits
    row = int(pos[0])                                   # and the rows themselves, one of them in float64
    x = (q[:, :, row].double().view(B, Hkv, Hq // Hkv, 1, d) * k.double()[:, :, None, :row + 1]).sum(-1) / d ** 0.5
    assert torch.allclose(lse[:, :, row].double(), torch.logsumexp(x, -1).view(B, Hq), atol=1e-4, rtol=0)


def causal_reference(q, k, v):
    """Attention and log-normalisers in float64."""
    G, L, d = q.shape[1] // k.shape[1], q.shape[2], q.shape[3]
    x = torch.matmul(q.double(), k.double().repeat_interleave(G, 1).transpose(-1, -2).contiguous()) / d ** 0.5
    x = x.masked_fill(torch.ones(L, L, dtype=torch.bool, device=DEV).triu(1), float("-inf"))
    return torch.matmul(torch.softmax(x, -1), v.double().repeat_interleave(G, 1)), torch.logsumexp(x, -1)


# fp32 calls by the 16-row kernel (at most 512 workgroups for 64 channels, 256 for 128; twice that from 512 rows on, for 64 channels up
# to 14 heads, or 1000 workgroups up to 20) - edges of its row and key blocks, one to nine key blocks for eight waves - and just past its rule
@pytest.mark.parametrize("d,B,Hq,Hkv,L", [
    (64, 1, 1, 1, 1), (64, 1, 3, 1, 15), (64, 2, 4, 2, 16), (64, 1, 5, 5, 17), (64, 1, 8, 2, 31), (64, 1, 8, 8, 33), (64, 3, 2, 1, 255),
    (64, 1, 4, 4, 257), (64, 1, 8, 8, 289), (64, 2, 16, 16, 256), (64, 2, 16, 16, 257), (64, 1, 8, 8, 2048), (64, 1, 8, 4, 2049),
    (64, 1, 14, 7, 1168), (64, 1, 14, 7, 1169), (64, 2, 8, 4, 992), (64, 1, 16, 4, 993), (64, 1, 20, 4, 800), (64, 1, 21, 7, 512), (64, 4, 8, 8, 512),
    (128, 1, 2, 1, 7), (128, 1, 4, 2, 47), (128, 1, 16, 4, 256), (128, 1, 16, 4, 257), (128, 1, 8, 2, 1000), (128, 1, 8, 2, 1025)])
def test_fp32_calls_of_few_rows(d, B, Hq, Hkv, L):
    g = torch.Generator(device=DEV).manual_seed(L + d)
    q = torch.randn(B, L, Hq, d, generator=g, device=DEV).transpose(1, 2)          # rows of a head apart by the others
    k, v = (torch.randn(B, Hkv, L, d, generator=g, device=DEV) for _ in range(2))
    k[..., ::17] *= 15.0
    out, lse, _ = zb.zc_prefill_attention(q, k, v)
    want, want_lse = causal_reference(q, k, v)
    # A logit is an fp32 sum of up to 128 products, of magnitudes that sum up to 2^8 here: off by a few 2^-16 at
    # the most, and so is a weight, relatively; the sums over keys average such errors.
    assert (out.double() - want).abs().max() < 1e-4 and (lse.double() - want_lse).abs().max() < 1e-4


def test_fp32_key_blocks_of_minus_infinity():
    """Blocks of 32 keys whose logits are all -inf, as many as a wave of the 16-row kernel has: weight 0."""
    B, H, L, d = 1, 4, 300, 64
    g = torch.Generator(device=DEV).manual_seed(5)
    q, k, v = (torch.randn(B, H, L, d, generator=g, device=DEV) for _ in range(3))
    q[..., 3] = 1.0
    k[:, :, 160:192] = 0.0
    k[:, :, 160:192, 3] = float("-inf")
    out, lse, _ = zb.zc_prefill_attention(q, k, v)
    want, want_lse = causal_reference(q, k, v)
    assert (out.double() - want).abs().max() < 1e-4 and (lse.double() - want_lse).abs().max() < 1e-4
