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


@pytest.mark.parametrize("special", [False, True])
@pytest.mark.parametrize("H,D,dtype,k,bits", [
    (1, 64, torch.bfloat16, 1, (4, 2)), (1, 64, torch.float32, 128, (2, 4)),          # rows of half the lanes keys take
    (3, 64, torch.float16, 17, (8, 2)), (4, 64, torch.bfloat16, 128, (4, 2)),         # four teams a workgroup
    (5, 64, torch.float32, 33, (2, 8)), (8, 64, torch.float16, 65, (4, 2)),           # two
    (12, 64, torch.bfloat16, 96, (4, 2)), (12, 64, torch.float16, 97, (2, 4)),        # eight keys a thread, and one too many
    (8, 128, torch.bfloat16, 90, (2, 4)), (8, 128, torch.float16, 91, (4, 2)),        # the most bytes, and one token more
    (8, 128, torch.float32, 45, (4, 2)), (16, 128, torch.bfloat16, 45, (2, 8)), (16, 128, torch.float32, 22, (4, 2)),
])
def test_short_subsets_as_beside_long_ones(H, D, dtype, k, bits, special):
    """A subset short enough for the one-launch kernel, alone, and the same beside one too long for it, which takes the
    kernels of longer calls: all that belongs to the short one bit for bit, in joint and single calls, from token-major
    tensors; the other, empty one has its default parameters.  (special: zeros, infinities, NaN, a channel of nothing else.)"""
    B, n = 3, 131
    g = torch.Generator(device=DEV).manual_seed(H + k)
    X, Y = ((3 * torch.randn(B, k + n, H, D, generator=g, device=DEV)).to(dtype).permute(0, 2, 1, 3) for _ in range(2))
    order = torch.stack([torch.randperm(k + n, generator=g, device=DEV) for _ in range(B)]).int()
    sal, reg = (t.sort(dim=1).values.contiguous() for t in (order[:, :k], order[:, k:]))
    if special:
        first, last = sal[1, 0].item(), sal[1, -1].item()
        for T in (X, Y):
            T[0, 0, :, 1] = 0.0
            T[0, 0, :, 2] = -0.0
            T[1, 0, first, 3] = float("inf")
            T[1, 0, last, 4] = -float("inf")
            T[1, H - 1, first, D - 1] = float("nan")
            T[2, H - 1, :, D - 2] = float("nan")
    forms = [("channel", zb.ZC_LAYOUT_ROW), ("cst", zb.ZC_LAYOUT_TGROUP)]
    want, got, one = ([_packed(f, B, H, D, k, n, bits) for f in forms] for _ in range(3))
    none = reg[:, :0]
    zb.zc_quantize_pack_kv(X, Y, sal, reg, *want, pos_offset=7)
    zb.zc_quantize_pack_kv(X, Y, sal, none, *got, pos_offset=7)
    zb.zc_quantize_pack(X, sal, none, one[0], pos_offset=7)
    zb.zc_quantize_pack(Y, sal, none, one[1], pos_offset=7)
    raw = lambda t: t.contiguous().view(torch.uint8)
    for w, *others in zip(want, got, one):
        for o in others:
            for name in ("codes_hi", "tok_scale_hi", "tok_zero_hi", "pos_hi"):
                a, b = getattr(w, name), getattr(o, name)
                if a is not None and name.startswith(("tok", "pos")):
                    a, b = a[:, :k], b[:, :k]
                assert a is None or torch.equal(raw(a), raw(b)), (w.scheme, name)
            for name, default in (("chan_scale", 1.0), ("chan_zero", 0.0)):
                a, b = getattr(w, name).flatten(), getattr(o, name).flatten()
                half = a.numel() // 2
                assert torch.equal(raw(a[:half]), raw(b[:half])), (w.scheme, name)
                assert bool((b[half:] == default).all()), (w.scheme, name)
            assert o.chunk_table.flatten()[:4].tolist() == [0, k, 0, 0] and o.chunks == [(0, k, 0, 0)]


@pytest.mark.parametrize("B,H,D,k,n,dtype", [
    (40, 8, 128, 90, 90, torch.bfloat16), (12, 8, 64, 90, 90, torch.float32), (130, 4, 64, 60, 60, torch.float32),      # past what workgroups may read
    (64, 4, 128, 22, 90, torch.float16), (64, 8, 128, 11, 45, torch.bfloat16),                                          # past it, of few readings a byte
    (31, 16, 128, 7, 30, torch.bfloat16), (33, 16, 128, 7, 30, torch.bfloat16),                                         # either side of half a workgroup a CU
    (64, 4, 64, 97, 97, torch.float16), (96, 4, 64, 97, 97, torch.float16), (129, 4, 64, 32, 32, torch.float32),        # keys alone: 256 and 384 workgroups, 516
])
def test_short_subsets_of_many_prompts(B, H, D, k, n, dtype):
    """Short subsets of a batch, which take the one launch or two by what its workgroups would read together, and each
    prompt in a call of its own: the same bits, in joint and single calls."""
    g = torch.Generator(device=DEV).manual_seed(B + n)
    X, Y = ((3 * torch.randn(B, H, k + n, D, generator=g, device=DEV)).to(dtype) for _ in range(2))
    sal, reg = zb.zc_select_salient(torch.rand(B, k + n, generator=g, device=DEV), k)
    forms = [("channel", zb.ZC_LAYOUT_ROW), ("cst", zb.ZC_LAYOUT_TGROUP)]
    joint, single = ([_packed(f, B, H, D, k, n, (4, 2)) for f in forms] for _ in range(2))
    zb.zc_quantize_pack_kv(X, Y, sal, reg, *joint, pos_offset=7)
    for x, p in zip((X, Y), single):
        zb.zc_quantize_pack(x, sal, reg, p, pos_offset=7)
    for b in (0, B // 2, B - 1):
        one = [_packed(f, 1, H, D, k, n, (4, 2)) for f in forms]
        zb.zc_quantize_pack_kv(X[b:b + 1], Y[b:b + 1], sal[b:b + 1], reg[b:b + 1], *one, pos_offset=7)
        for which, want in enumerate(one):
            for p in (joint[which], single[which]):
                for name in ARRAYS[:-1]:
                    a, w = getattr(p, name), getattr(want, name)
                    a = a.view(2, B, H * D)[:, b] if name.startswith("chan") else a.view(B, -1)[b]
                    assert torch.equal(a.flatten(), w.flatten()), (which, b, name)


@pytest.mark.parametrize("n", [20, 131])
@pytest.mark.parametrize("dtype", [torch.float16, torch.float32])
def test_channel_parameters_at_any_float(dtype, n):
    """Channel parameters are written where they are put, also at addresses that four bytes divide and sixteen do not (by
    the kernel of short subsets and those of longer ones): the same bits, and the floats beside them left alone."""
    B, H, D, k = 2, 3, 64, 5
    g = torch.Generator(device=DEV).manual_seed(n)
    X, Y = (torch.randn(B, H, k + n, D, generator=g, device=DEV).to(dtype) for _ in range(2))
    sal, reg = zb.zc_select_salient(torch.rand(B, k + n, generator=g, device=DEV), k)
    forms = [("channel", zb.ZC_LAYOUT_ROW), ("cst", zb.ZC_LAYOUT_TGROUP)]
    want = [_packed(f, B, H, D, k, n, (4, 2)) for f in forms]
    zb.zc_quantize_pack_kv(X, Y, sal, reg, *want)
    for off in (1, 2, 3):
        got = [_packed(f, B, H, D, k, n, (4, 2)) for f in forms]
        wide = [[torch.full((a.numel() + 8,), -7.0, device=DEV) for a in (p.chan_scale, p.chan_zero)] for p in got]
        for p, (scale, zero) in zip(got, wide):
            p.c.chan_scale, p.c.chan_zero = scale[off:].data_ptr(), zero[off:].data_ptr()
        zb.zc_quantize_pack_kv(X, Y, sal, reg, *got)
        for w, p, arrays in zip(want, got, wide):
            assert torch.equal(w.codes_hi, p.codes_hi) and torch.equal(w.codes_lo, p.codes_lo)
            for a, b in zip((w.chan_scale, w.chan_zero), arrays):
                assert torch.equal(b[off:off + a.numel()], a.flatten())
                assert bool((b[:off] == -7.0).all()) and bool((b[off + a.numel():] == -7.0).all())


def _largest(form, H, n, bits, dtype):
    """`n` tokens of which a few are not zero, packed; the same few (and a zero one) in a call of their own."""
    D = 64
    x = torch.zeros(1, 1, n, D, dtype=dtype, device=DEV)
    rows = [0, 5, n // 2, n - 4096, n - 4095, n - 1]
    for r in rows:
        x[0, 0, r] = torch.arange(D, device=DEV) - 9 * (r % 3)
    rows.append(1)
    few = torch.cat([x[:, :, r:r + 1] for r in rows], 2)
    none = torch.empty(1, 0, dtype=torch.int32, device=DEV)
    out = []
    for t in (x, few):
        p = zb.PackedTensor(1, H, D, 0, t.shape[2], 8, bits, *form, max_chunks=1, device=DEV)
        zb.zc_quantize_pack(t.expand(1, H, -1, D), none, torch.arange(t.shape[2], dtype=torch.int32, device=DEV)[None], p)
        out.append(p)
    assert torch.equal(out[0].pos_lo[0, rows].cpu(), torch.tensor(rows, dtype=torch.int32))
    return rows, out


def test_values_of_more_threads_than_a_launch_counts():
    """A word group of four 8-bit codes takes a wave of k_pack_kv, so that 2^28 tokens reach 2^32 threads."""
    rows, (many, few) = _largest(("cst", zb.ZC_LAYOUT_TGROUP), 1, (1 << 28) + 4096, 8, torch.float16)

    def codes(p, slot):                               # blocks of 16 slots, 4 words of 64 channels, 4 slots a word
        return (p.codes_lo.view(torch.int32).view(-1, 4, 64)[slot // 16, slot % 16 // 4] >> (8 * (slot % 4))) & 0xff
    for i, r in enumerate(rows):
        assert torch.equal(many.tok_scale_lo[0, r], few.tok_scale_lo[0, i]) and torch.equal(many.tok_zero_lo[0, r], few.tok_zero_lo[0, i]), r
        assert torch.equal(codes(many, r), codes(few, i)), r


def test_keys_of_more_threads_than_a_launch_counts():
    """Four tokens of 8192 channels take 1024 threads, so that 2^24 tokens reach 2^32 (all heads read one)."""
    rows, (many, few) = _largest(("channel", zb.ZC_LAYOUT_ROW), 128, (1 << 24) + 4096, 2, torch.bfloat16)
    assert torch.equal(many.chan_scale, few.chan_scale) and torch.equal(many.chan_zero, few.chan_zero)
    a, b = many.codes_lo.view(128, -1, 16), few.codes_lo.view(128, -1, 16)
    for i, r in enumerate(rows):
        assert torch.equal(a[:, r], b[:, i]), r


@pytest.mark.parametrize("kind", ["tame", "nan", "wild"])
@pytest.mark.parametrize("n", [1, 2, 60, 61, 63, 517, 2600, 4096, 4097, 7003])
def test_two_bit_fp16_keys_by_thresholds(n, kind):
    """2-bit codes of fp16 keys that stay in registers, found by three thresholds a channel, against those
    of the kernel that divides every value (another layout, so another path): the same codes where
    values are ties of the rounding and one number beside them, equal, zeros of both signs, subnormal,
    the largest, far from zero in a narrow range, a NaN, or of a range without thresholds.  (Up to
    8 rows a thread divide too: 4096 tokens are the most that do, 4097 the fewest that do not.  Up to 60 take the one launch of
    short subsets, which divides.)"""
    from tests.pipeline_check import packed_to_chunks
    H, D = 3, 64
    g = torch.Generator().manual_seed(n)
    X = torch.randn(1, H, n, D, generator=g)
    steps = torch.randint(0, 7, (H, n), generator=g).float()
    at = lambda ch, x: X[0, :, :, ch].copy_(x)
    for i, scale in enumerate((1.0, 0.75, 3.1, 2.0 ** -14, 2.0 ** -22, 9000.0)):
        at(i, scale * steps / 2)                                                            # every half step: ties
        at(8 + i, (scale * steps / 2).half().view(torch.int16).add((steps % 3 - 1).short() * (steps > 0)).view(torch.float16).float())
        at(16 + i, scale * (steps / 2 - 1.7))                                               # a zero point between
    at(24, torch.full((H, n), 0.3))
    at(25, torch.zeros(H, n))
    at(26, torch.where(steps > 3, 0.0, -0.0))
    at(27, torch.where(steps > 3, 65504.0, -65504.0))
    at(28, 1000.0 + steps / 2)
    at(29, -3.0 - steps * 2.0 ** -8)
    at(30, 2.0 ** -24 * (steps - 3))
    X = X.to(torch.float16)
    if kind == "nan":
        X[0, 0, n // 2, 5] = X[0, 2, 0, 63] = float("nan")
    if kind == "wild":
        X[0, 1, n // 2, 33] = float("inf")
        X[0, 2, 0, 12] = -float("inf")
    X = X.to(DEV)
    idx = torch.arange(n, dtype=torch.int32, device=DEV)[None]
    none = idx[:, :0]
    got = []
    for layout in (zb.ZC_LAYOUT_ROW, zb.ZC_LAYOUT_TGROUP):
        p = _packed(("channel", layout), 1, H, D, 64, zb.load().zc_arena_slots(n, 1), (4, 2))
        zb.zc_quantize_pack(X, none, idx, p)
        got.append((torch.as_tensor(packed_to_chunks(p, [0])[0].lo.codes), p.chan_scale.clone(), p.chan_zero.clone()))
    (row, *params), (tgroup, *want) = got
    assert all(torch.equal(a.view(torch.int32), b.view(torch.int32)) for a, b in zip(params, want))
    assert torch.equal(row, tgroup), (row != tgroup).nonzero()[:8]


@pytest.mark.parametrize("dtype", [torch.float16, torch.bfloat16, torch.float32])
@pytest.mark.parametrize("layout", [zb.ZC_LAYOUT_ROW, zb.ZC_LAYOUT_TGROUP])
@pytest.mark.parametrize("n", [1, 9, 32, 61, 130, 1000, 9000, 40000])
def test_keys_of_a_channel_of_nan(n, layout, dtype):
    """A channel that is all NaN has NaN for its parameters, whether its tokens stay in registers (of the one launch of
    short subsets up to 32 in fp32 and 60, of the column sweep from 61 on), come in
    batches or in ranges, whatever part of the workgroup they leave without a row; the other channels have theirs."""
    H, D = 2, 64
    X = torch.randn(1, H, n, D, generator=torch.Generator().manual_seed(n)).to(dtype)
    X[0, 0, n // 2, 3] = 0.25
    X[0, 0, n // 3, 3] = float("nan") if n > 1 else 0.25
    X[0, 1, :, 7] = float("nan")
    idx = torch.arange(n, dtype=torch.int32, device=DEV)[None]
    p = _packed(("channel", layout), 1, H, D, 64, zb.load().zc_arena_slots(n, 1), (4, 2))
    zb.zc_quantize_pack(X.to(DEV), idx[:, :0], idx, p)
    nan = torch.zeros(H * D, dtype=torch.bool)
    nan[D + 7] = True
    for a in (p.chan_scale, p.chan_zero):
        low = a.flatten()[-H * D:].cpu()                    # (the subset of few bits is the second)
        assert torch.equal(low.isnan(), nan) and not bool(low.isinf().any())


@pytest.mark.parametrize("cap", [524224, 524288])
def test_keys_on_either_side_of_4_gigabytes(cap):
    """Codes of a batch element just below and at 2^32 bytes: the first still have 32-bit offsets in the column
    sweep, the second take the way of keys that do not stay in registers; either has the codes of a small arena.  (130
    tokens: more than the one launch of short subsets takes, whose offsets have 64 bits.)"""
    H, D, n = 64, 128, 130
    X = torch.randn(1, H, 2 * n, D, generator=torch.Generator().manual_seed(cap)).to(torch.bfloat16).to(DEV)
    idx = torch.arange(n, dtype=torch.int32, device=DEV)[None]
    got = []
    for c in (cap, 384):
        p = zb.PackedTensor(1, H, D, 64, c, 2, 8, "channel", zb.ZC_LAYOUT_ROW, max_chunks=2, device=DEV)
        for x in (X[:, :, :n], X[:, :, n:]):                    # (the second chunk begins at slot 192)
            zb.zc_quantize_pack(x, idx[:, :0], idx, p)
        rows = p.codes_lo.view(H, c, D)
        assert not bool(rows[:, n:192].any()) and not bool(rows[:, 192 + n:384].any())
        got.append((torch.cat([rows[:, :n], rows[:, 192:192 + n]], 1).clone(), p.chan_scale[:2].clone(), p.chan_zero[:2].clone()))
        del p, rows
    assert all(torch.equal(a, b) for a, b in zip(*got))
