"""Prefill attention: the probe rows' normalisers, from the attention kernel itself and by a launch of their own."""
import pytest
import torch

from paper_2405_14256_amd import binding as zb

pytestmark = pytest.mark.gpu
DEV = "cuda"


# (dtype, d, B, Hq, Hkv, L, P): up to two probes a thread come from the kernel - workgroups of 64, 128 and
# 256 threads (fp32, by heads and length), 256 and 512 (16 bit) - one more takes the other launch
@pytest.mark.parametrize("dtype,d,B,Hq,Hkv,L", [(torch.float32, 64, 1, 3, 1, 97), (torch.float32, 64, 2, 160, 160, 250),
                                                (torch.float32, 128, 1, 128, 32, 800), (torch.float16, 128, 2, 4, 2, 391),
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
