"""Decode over caches with 8-bit codes: blocks of 16 slots, codes of every width as exact centred fp16 numbers."""
import pytest
import torch

from paper_2405_14256_amd import binding as zb

pytestmark = pytest.mark.gpu
DEV = "cuda"


@pytest.mark.parametrize("q_scale,v_scale", [(1.0, 1.0), (8.0, 50.0), (1 / 64, 1e-3)])
@pytest.mark.parametrize("bits", [(8, 8), (8, 4), (8, 2), (2, 8), (4, 8)])
@pytest.mark.parametrize("dtype,d,B,Hkv,G", [(torch.float32, 128, 1, 2, 4), (torch.float32, 64, 2, 1, 8), (torch.bfloat16, 128, 2, 3, 1),
                                             (torch.float16, 64, 70, 4, 2), (torch.float16, 128, 64, 5, 4)])
def test_decode_with_8_bit_codes(bits, dtype, d, B, Hkv, G, q_scale, v_scale):
    """Segments that end at, before and after a block's edge, empty subsets, every scheme on
    either tensor, launches below and above one workgroup per compute unit, outlier key channels,
    queries and values over three orders of magnitude, against attention in float64 over the
    de-quantized cache."""
    g = torch.Generator().manual_seed(d * B + bits[0])
    lib = zb.load()
    sizes = [(33, 47), (16, 15), (0, 17), (1, 0), (64, 64)]
    T = 19
    n = sum(a + b for a, b in sizes)
    X = torch.randn(2, B, Hkv, n + T, d, generator=g)
    X[0, ..., ::21] *= 15.0
    X[1] *= v_scale
    X = X.to(dtype).to(DEV)
    q = ((torch.randn(B, Hkv * G, d, generator=g) + 0.25) * q_scale).to(dtype).to(DEV)
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
        # Errors as root mean squares over all heads.  A logit is a sum of d products of the query, held
        # to 22 bits, with centred codes: off by a few 2^-22 of the logits' spread; the normaliser also
        # carries its own rounding, and a weight (so an output) is off by as much as its logit, relatively.
        spread = float(logits.square().mean().sqrt())
        err_lse = float((lse.double() - want_lse).square().mean().sqrt())
        assert err_lse <= 2.0 ** -19 * spread + 2.0 ** -22 * float(want_lse.abs().max()), (k_scheme, v_scheme, err_lse, spread)
        # 16-bit results: the rounding of the result itself, 2^-12 (fp16) or 2^-9 (bf16) over the square
        # root of 3 times a mean of about 1.5; of fp16 values near 1e-4 (spacing 2^-24) up to 3.1e-4.
        # (Measured: fp16 2.1e-4 and 3.04e-4, bf16 1.8e-3; with single fp16 weights fp16 5.9e-4.)
        err = float((out.double() - want).norm() / want.norm())
        tol = {torch.float32: 1e-6 + 4e-7 * spread, torch.float16: 2.3e-4 if v_scale >= 1 else 3.3e-4, torch.bfloat16: 2e-3}[dtype]
        assert err <= tol, (k_scheme, v_scheme, err, spread)


def workgroups_of_a_head(B, Hkv, d, sizes, T, bits, cus=256):
    """What a launch chooses from for a cache of one chunk: (cost units of a head, its workgroups where a CU has two, where it
    has one, whether the latter are taken), or None where all workgroups of the finest split fit one per CU."""
    ceil = lambda a, b: -(-a // b)
    units = sum(ceil(n, 16 if b == 8 else 32) + 3 for n, b in zip(sizes, bits) if n)
    heads, finest = B * Hkv, min(ceil(units, 8), 32)
    if heads * finest <= cus:
        return None
    two = min(range(1, finest + 1), key=lambda c: ceil(heads * c, 2 * cus) * (48 + ceil(units, c)))
    one, tail = cus // heads, 2 * ceil(T, 16) + 3
    lone = ((21, 20, 19), (19, 17, 16), (23, 22, 20))[2 if one == 1 else d == 128][bits.count(8)]
    gain = 12 if one == 1 else 2
    return units, two, one, 0 < one < two and lone * ceil(units + tail, one) <= 32 * (gain + ceil(units + tail, two))


# Pairs on either side of the rule, at both head widths and every number of 8-bit widths; a head with two workgroups, where one
# of a CU leaves a third of the chip idle; a head to a workgroup; 12 heads, which two only give half the CUs; too few units to ask;
# more heads than CUs
@pytest.mark.parametrize("B,Hkv,d,L,bits,one", [
    (2, 8, 128, 10300, (4, 2), True), (2, 8, 128, 12800, (4, 2), False), (8, 8, 128, 2200, (4, 4), True), (8, 8, 128, 2900, (4, 4), False),
    (2, 8, 64, 7600, (4, 2), True), (2, 8, 64, 10400, (2, 4), False), (4, 8, 128, 13400, (8, 4), True), (4, 8, 128, 20000, (8, 4), False),
    (4, 8, 64, 3000, (8, 2), True), (4, 8, 64, 3600, (2, 8), False), (8, 8, 64, 1300, (8, 8), True), (8, 8, 64, 1500, (8, 8), False),
    (16, 8, 128, 3000, (8, 8), True), (10, 9, 64, 400, (8, 4), True), (10, 9, 64, 700, (8, 4), False), (43, 2, 128, 800, (2, 2), True),
    (43, 2, 128, 1000, (2, 2), False), (25, 8, 64, 1100, (4, 2), True), (25, 8, 64, 1700, (4, 2), False), (31, 8, 128, 900, (8, 8), True),
    (43, 4, 128, 1500, (8, 8), False), (1, 12, 64, 9000, (2, 8), True), (3, 12, 128, 1300, (4, 4), None), (100, 3, 128, 300, (4, 2), False),
    (2, 8, 128, 8000, (4, 2), True), (2, 8, 128, 8400, (4, 2), True), (4, 8, 128, 7901, (8, 4), True), (4, 8, 128, 8300, (8, 4), True),
    (8, 8, 128, 700, (8, 4), True), (8, 8, 128, 2000, (8, 4), True)])
def test_decode_with_one_or_two_workgroups_a_cu(B, Hkv, d, L, bits, one):
    """Either side of the rule by which a launch takes one workgroup per compute unit: every sequence
    of a batch of equal ones has the answer that it has alone, but for the order of the partial sums."""
    G, T = 2, 37
    rule = workgroups_of_a_head(B, Hkv, d, (L // 5, L - L // 5), T, bits)
    assert one == (rule and rule[3]), rule
    g = torch.Generator().manual_seed(L)
    lib = zb.load()
    X = torch.randn(2, 1, Hkv, L + T, d, generator=g).to(DEV)
    q = torch.randn(1, Hkv * G, d, generator=g).to(DEV)
    scores = torch.rand(1, L, generator=g).to(DEV)
    k = L // 5
    res = []
    for n in (1, B):
        K, V = (x.expand(n, -1, -1, -1).contiguous() for x in X)
        sal, reg = zb.zc_select_salient(scores.expand(n, -1).contiguous(), k)
        mk = lambda s, layout: zb.PackedTensor(n, Hkv, d, lib.zc_arena_slots(k, 1), lib.zc_arena_slots(L - k, 1), *bits, s, layout, max_chunks=1, device=DEV)
        Kp, Vp = mk("channel", zb.ZC_LAYOUT_ROW), mk("cst", zb.ZC_LAYOUT_TGROUP)
        zb.zc_quantize_pack(K[:, :, :L], sal, reg, Kp)
        zb.zc_quantize_pack(V[:, :, :L], sal, reg, Vp)
        lse = torch.empty(n, Hkv * G, dtype=torch.float32, device=DEV)
        out = zb.zc_decode_attention(q.expand(n, -1, -1).contiguous(), Kp, Vp, K[:, :, L:], V[:, :, L:], T, lse_out=lse)
        res.append((out, lse))
    (alone, lse1), (out, lse) = res
    assert torch.equal(out, out[:1].expand_as(out)) and torch.equal(lse, lse[:1].expand_as(lse))
    # A sum of L weights of at most a few units in chains of L / 32 and more: each term is off by 2^-24 of the
    # sum so far, which adds up like a random walk - 2^-24 sqrt(L) - times what the values' spread leaves.
    # Either order has this error; four times both is 2^-21 sqrt(L) of the largest output.
    tol = 2.0 ** -21 * L ** 0.5
    assert float((lse - lse1).abs().max()) <= tol
    assert float((out - alone).abs().max()) <= tol * max(1.0, float(alone.abs().max()))
