"""zc_quantize_pack_kv over every pair of scheme and layout its two tensors may have, in either
place, below and above the sizes at which channelwise keys stay in registers: every array as two
zc_quantize_pack calls leave it, bit for bit.  All arrays start as a pattern, so that a tensor
that is not packed shows."""
import pytest
import torch

from paper_2405_14256_amd import binding as zb

pytestmark = pytest.mark.gpu
DEV = "cuda"

FORMS = [(s, l) for s in ("channel", "cst", "token") for l in (zb.ZC_LAYOUT_ROW, zb.ZC_LAYOUT_TGROUP)]
ARRAYS = ("codes_hi", "codes_lo", "tok_scale_hi", "tok_zero_hi", "tok_scale_lo", "tok_zero_lo", "pos_hi", "pos_lo",
          "chan_scale", "chan_zero", "chunk_table")


def _packed(form, B, H, D, k, n, bits):
    p = zb.PackedTensor(B, H, D, k, n, *bits, *form, max_chunks=1, device=DEV)
    for name in ARRAYS:
        getattr(p, name).fill_(0x5A)
    return p


def _compare(first, second, B, H, D, k, n, dtype, bits=(4, 2)):
    g = torch.Generator(device=DEV).manual_seed(H + n)
    X, Y = ((3 * torch.randn(B, H, k + n, D, generator=g, device=DEV)).to(dtype) for _ in range(2))
    order = torch.stack([torch.randperm(k + n, generator=g, device=DEV) for _ in range(B)]).int()
    sal, reg = (t.sort(dim=1).values.contiguous() for t in (order[:, :k], order[:, k:]))
    want, got = ([_packed(f, B, H, D, k, n, bits) for f in (first, second)] for _ in range(2))
    zb.zc_quantize_pack(X, sal, reg, want[0], pos_offset=7)
    zb.zc_quantize_pack(Y, sal, reg, want[1], pos_offset=7)
    zb.zc_quantize_pack_kv(X, Y, sal, reg, *got, pos_offset=7)
    for which, (a, b) in enumerate(zip(want, got)):
        assert a.chunks == b.chunks and (a.c.n_hi, a.c.n_lo, a.c.n_chunks) == (b.c.n_hi, b.c.n_lo, b.c.n_chunks)
        for name in ARRAYS:
            assert torch.equal(getattr(a, name), getattr(b, name)), (first, second, which, name)
    # (the pattern is gone where a token's positions and parameters belong: packed, not both left alone)
    for p in got:
        assert torch.equal(p.pos_hi[:, :k], sal + 7) and torch.equal(p.pos_lo[:, :n], reg + 7)
        if p.scheme != "channel":
            assert bool((p.tok_scale_lo[:, :n] != 0x5A).all())


@pytest.mark.parametrize("second", FORMS)
@pytest.mark.parametrize("first", FORMS)
@pytest.mark.parametrize("B,H,D,k,n,dtype,bits", [
    (2, 8, 128, 70, 131, torch.bfloat16, (4, 2)),       # rows of a workgroup's width
    (1, 40, 128, 33, 90, torch.float16, (8, 4)),        # rows that go through the kernel of wide values
    (1, 10, 128, 65, 97, torch.float32, (2, 8)),
])
def test_every_pair_of_forms(first, second, B, H, D, k, n, dtype, bits):
    _compare(first, second, B, H, D, k, n, dtype, bits)


# Subsets that do not stay in registers: too long for the widest workgroup, or (16-bit rows of more
# than 512 channels) only in slices of 16 channels.
@pytest.mark.parametrize("first", [("channel", zb.ZC_LAYOUT_ROW), ("cst", zb.ZC_LAYOUT_TGROUP), ("token", zb.ZC_LAYOUT_ROW)])
@pytest.mark.parametrize("H,D,n,dtype", [(1, 64, 10300, torch.float16), (8, 128, 5200, torch.bfloat16), (1, 128, 5200, torch.float32),
                                         (20, 128, 2600, torch.float16)])
def test_channelwise_rows_in_second_place(first, H, D, n, dtype):
    _compare(first, ("channel", zb.ZC_LAYOUT_ROW), 1, H, D, 40, n, dtype)
