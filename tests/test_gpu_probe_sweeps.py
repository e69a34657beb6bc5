"""Probe saliency: how the row blocks of the first sweep share a head's workgroups, tile edges of both sweeps."""
import ctypes as C

import pytest
import torch

from paper_2405_14256_amd import binding as zb

pytestmark = pytest.mark.gpu
DEV = "cuda"


def reference(q, k, rows, pos, lse=None):
    """Eq. 9 + Eq. 8 in float64 on the GPU, a head at a time."""
    B, Hq, _, d = q.shape
    G, Lk = Hq // k.shape[1], k.shape[2]
    seen = pos[:, None] >= torch.arange(Lk, device=DEV)[None]
    count = seen.sum(0).double()
    scores = torch.zeros(B, Lk, dtype=torch.float64, device=DEV)
    for b in range(B):
        for h in range(Hq):
            x = q[b, h, rows].double() @ k[b, h // G].double().T / d ** 0.5
            x = x.masked_fill(~seen, float("-inf"))
            norm = torch.logsumexp(x, -1) if lse is None else lse[b, h].double()
            scores[b] += torch.exp(x - norm[:, None]).sum(0) / count.clamp(min=1)
    return scores / Hq


# (B, Hq, Hkv, d, L, dtype, probe positions): one row block and several ranges, blocks that see
# from one tile to all of them, a block of one row, rows below a tile's width, more ranges than a
# block may have, more than 64 blocks, both halves of a tile masked, the last tile ragged
def spread(L, P):
    return torch.linspace(0, L - 1, P).round().long().unique()


CASES = [
    (1, 1, 1, 128, 33000, torch.bfloat16, lambda L: spread(L, 40)),
    (1, 8, 2, 128, 4097, torch.bfloat16, lambda L: spread(L, 385)),
    (2, 6, 3, 64, 2111, torch.float16, lambda L: spread(L, 129)),
    (1, 4, 4, 64, 1025, torch.float32, lambda L: torch.cat([torch.arange(200), torch.tensor([1024])])),
    (1, 2, 1, 128, 777, torch.float32, lambda L: torch.arange(L - 300, L)),
    (3, 5, 5, 128, 191, torch.float16, lambda L: torch.arange(60, 190)),
    (1, 1, 1, 64, 8400, torch.bfloat16, lambda L: torch.arange(L - 8300, L)),
    (1, 40, 40, 64, 130, torch.bfloat16, lambda L: torch.arange(L)),
    (1, 16, 4, 128, 2000, torch.float32, lambda L: torch.arange(L - 200, L)),        # two blocks that see all but the same columns
    (2, 200, 200, 64, 300, torch.bfloat16, lambda L: spread(L, 30)),                  # a single block of more heads than get two ranges
    (1, 130, 130, 64, 200, torch.float32, lambda L: spread(L, 33)),                   # of four tiles at most: one range
    (1, 8, 2, 128, 4500, torch.float32, lambda L: spread(L, 450)),                    # whole rounds of workgroups a CU
    # last blocks of up to 32, of 33 to 64 and of 65 rows; the most probes looked up from LDS at once and one more, some in
    # front of the last columns, some behind the first; heads enough for a full chip of blocks of different lengths
    (1, 4, 2, 128, 1500, torch.bfloat16, lambda L: spread(L, 160)),
    (1, 4, 2, 64, 1500, torch.float32, lambda L: spread(L, 161)),
    (1, 4, 2, 128, 1500, torch.float16, lambda L: spread(L, 192)),
    (2, 4, 2, 64, 1500, torch.bfloat16, lambda L: spread(L, 193)),
    (1, 2, 1, 128, 3000, torch.bfloat16, lambda L: spread(L, 512)),
    (1, 2, 1, 128, 3000, torch.float32, lambda L: spread(L, 513)),
    (1, 2, 2, 64, 2600, torch.bfloat16, lambda L: torch.arange(L - 1100, L)),
    (1, 32, 8, 128, 2100, torch.bfloat16, lambda L: torch.cat([spread(L - 110, 110), torch.arange(L - 110, L)]).unique()),
    # more probes than are looked up at once: two halves of the table and a row, three, six and the last tile ragged, one that sees
    # the first columns only
    (1, 2, 1, 64, 2000, torch.float16, lambda L: torch.arange(L - 769, L)),
    (1, 3, 3, 128, 1600, torch.bfloat16, lambda L: torch.arange(1538)),
    (1, 2, 2, 64, 3000, torch.float32, lambda L: torch.cat([torch.arange(90), spread(L, 700)]).unique()),
    # few probes over several ranges, joined by sweep 2; as many ranges as two at a time leave of nine
    (10, 16, 4, 64, 352, torch.bfloat16, lambda L: spread(L, 18)),
    (3, 8, 8, 64, 900, torch.float16, lambda L: spread(L, 31)),
    (1, 2, 1, 64, 900, torch.bfloat16, lambda L: spread(L, 300)),
    # ranges joined by a launch: in front of the one launch of few probes, and of a sweep 2 of more than a round of workgroups
    (3, 12, 12, 64, 105, torch.float32, lambda L: spread(L, 10)),
    (36, 8, 4, 64, 700, torch.bfloat16, lambda L: spread(L, 70)),
]


@pytest.mark.parametrize("external", [False, True])
@pytest.mark.parametrize("case", range(len(CASES)))
def test_scores_of_row_blocks_and_ranges(case, external):
    B, Hq, Hkv, d, L, dtype, probes = CASES[case]
    g = torch.Generator(device=DEV).manual_seed(case)
    pos = probes(L).to(DEV)
    P = pos.numel()
    q = (torch.randn(B, Hq, P, d, generator=g, device=DEV) + 0.25).to(dtype)     # rows in an order of their own
    rows = torch.randperm(P, generator=g, device=DEV)
    k = torch.randn(B, Hkv, L, d, generator=g, device=DEV)
    k[..., ::31] *= 15.0
    k = k.to(dtype)
    lse = 40.0 + torch.randn(B, Hq, P, generator=g, device=DEV) if external else None
    want = reference(q, k, rows, pos, lse)
    per_head = torch.empty(B, Hq, L, device=DEV)
    for ph in (None, per_head):
        got = zb.zc_probe_saliency(q, k, pos.int(), probe_rows=rows.int(), lse_ext=lse, scores_per_head=ph)
        # A logit is an fp32 sum of up to 128 exact products: off by a few 2^-24 of the sum of their
        # magnitudes, at most about 2^8 here, so a probability by up to 2^-13 and, with errors of
        # either sign over many rows and heads, far less; measured 2e-6 at most.
        rel = ((got.double() - want).abs() / want.clamp(min=1e-30)).max().item()
        assert rel < 3e-5, (rel, ph is not None)
    assert torch.allclose(per_head.mean(1), got, rtol=1e-5, atol=0)


# Masked keys: columns whose logits are -inf, in tiles that a row sees in part, in whole tiles and as
# all of the columns that a row's lane sees of its first tiles.
@pytest.mark.parametrize("d,dtype,P", [(64, torch.float32, 40), (128, torch.bfloat16, 96), (64, torch.float16, 26)])
def test_scores_with_logits_of_minus_infinity(d, dtype, P):
    B, Hq, Hkv, L = 1, 4, 2, 300
    g = torch.Generator(device=DEV).manual_seed(P)
    pos = torch.cat([torch.arange(5, 12), torch.tensor([44, 70]), spread(L, 400)[-(P - 9):]]).unique().to(DEV)
    q = torch.randn(B, Hq, pos.numel(), d, generator=g, device=DEV)
    q[..., 3] = 1.0
    k = torch.randn(B, Hkv, L, d, generator=g, device=DEV)
    k[:, :, [0, 1, 2, 3, 8, 64, 65, 66, 67, 128]] = 0.0
    k[:, :, [0, 1, 2, 3, 8, 64, 65, 66, 67, 128], 3] = float("-inf")
    k[:, :, 32:64] = 0.0
    k[:, :, 32:64, 3] = float("-inf")
    q, k = q.to(dtype), k.to(dtype)
    rows = torch.arange(pos.numel(), device=DEV)
    got = zb.zc_probe_saliency(q, k, pos.int(), probe_rows=rows.int())
    want = reference(q, k, rows, pos)
    hidden = torch.isinf(k[0, 0, :, 3])
    assert bool((got[:, hidden] == 0).all()) and bool(torch.isfinite(got).all())
    rel = ((got.double() - want).abs() / want.clamp(min=1e-30))[:, ~hidden].max().item()
    assert rel < 3e-5, rel                       # (the bound of the test above)


# Columns 2^72 above all before them, in a tile that every row sees and in one that some rows see: the rows' references move
# while only terms are summed.  Blocks of one, two and both halves of a wave's rows.
@pytest.mark.parametrize("d,dtype,P", [(128, torch.bfloat16, 33), (64, torch.float16, 97), (128, torch.float32, 160), (128, torch.float16, 192)])
def test_scores_whose_references_move(d, dtype, P):
    B, Hq, Hkv, L = 1, 4, 2, 1500
    g = torch.Generator(device=DEV).manual_seed(P)
    pos = torch.cat([spread(800, 20) + 400, torch.arange(L - (P - 20), L)]).unique().to(DEV)
    q = torch.randn(B, Hq, pos.numel(), d, generator=g, device=DEV)
    q[..., 3] = 1.0
    k = torch.randn(B, Hkv, L, d, generator=g, device=DEV)
    k[..., 3] = 0.0
    k[:, :, [333, 777], 3] = torch.tensor([50.0, 100.0], device=DEV) * d ** 0.5
    q, k = q.to(dtype), k.to(dtype)
    rows = torch.arange(pos.numel(), device=DEV)
    got = zb.zc_probe_saliency(q, k, pos.int(), probe_rows=rows.int())
    want = reference(q, k, rows, pos)
    # (the bound of the first test: the terms of a logit sum up to less than 2^8)
    rel = ((got.double() - want).abs() / want.clamp(min=1e-30)).max().item()
    assert rel < 3e-5, rel


# A row's reference is a maximum of scaled logits: columns a lane does not see stay out of it for a negative scale too.
@pytest.mark.parametrize("case", [1, 2, 3, 4])
def test_scores_of_a_negative_scale(case):
    B, Hq, Hkv, d, L, dtype, probes = CASES[case]
    g = torch.Generator(device=DEV).manual_seed(case)
    pos = probes(L).to(DEV)
    q = torch.randn(B, Hq, pos.numel(), d, generator=g, device=DEV).to(dtype)
    k = torch.randn(B, Hkv, L, d, generator=g, device=DEV).to(dtype)
    rows = torch.arange(pos.numel(), dtype=torch.int32, device=DEV)
    got = zb.zc_probe_saliency(q, k, pos.int(), probe_rows=rows, sm_scale=-0.25)
    want = reference(q.double() * (-0.25 * d ** 0.5), k, rows.long(), pos)
    # (the bound of the first test: a logit's terms sum up to 0.25 * 128 * E|q k| = 21, below its 2^8; a matrix
    # instruction drops bits of products without regard to sign, so the scores of -q and 0.25 are not the same bits)
    rel = ((got.double() - want).abs() / want.clamp(min=1e-30)).max().item()
    assert rel < 3e-5, rel


# A workspace of the least size: the pairs of the column ranges have no place beside the per-head scores, and are joined in front of sweep 2.
@pytest.mark.parametrize("case", [1, 2, 12, 16, len(CASES) - 1])
def test_scores_in_the_least_workspace(case):
    B, Hq, Hkv, d, L, dtype, probes = CASES[case]
    g = torch.Generator(device=DEV).manual_seed(case)
    pos = probes(L).int().to(DEV)
    P = pos.numel()
    q = torch.randn(B, Hq, L, d, generator=g, device=DEV).to(dtype)
    k = torch.randn(B, Hkv, L, d, generator=g, device=DEV).to(dtype)
    want = zb.zc_probe_saliency(q, k, pos)
    least = -(-B * Hq * P * 68 // 256) * 256 + B * Hq * L * 4          # a log-sum-exp and eight pairs a row, the per-head scores
    lib = zb.load()
    assert least < lib.zc_probe_saliency_workspace(B, Hq, L, P)
    ws = torch.full((least + 64,), 0xff, dtype=torch.uint8, device=DEV)
    got = torch.empty_like(want)
    code = {torch.float32: zb.ZC_F32, torch.float16: zb.ZC_F16, torch.bfloat16: zb.ZC_BF16}[dtype]
    views = [zb.zc_tensor4(t.data_ptr(), code, 0, *t.shape, *t.stride()[:3]) for t in (q, k)]
    call = lambda n: lib.zc_probe_saliency(C.byref(views[0]), C.byref(views[1]), None, pos.data_ptr(), P, 0.0, None,
                                           got.data_ptr(), None, ws.data_ptr(), n, torch.cuda.current_stream().cuda_stream)
    assert call(least - 1) == -3
    assert call(least) == 0
    assert bool((ws[least:] == 0xff).all())
    # (the ranges may be cut elsewhere: sums of the same terms in another order, each sum off by a few 2^-24)
    assert torch.allclose(got, want, rtol=1e-5, atol=0)


# Heads that share an XCD's places in groups (a multiple of 8 heads, and so many tokens that fewer than an XCD's heads fill its
# places): groups of 2 and 2; 3 and 2; 3, 3 and 1; 4 and 3 of a batch element each; 3 and 2 on the border of two batch elements
@pytest.mark.parametrize("B,Hq,Hkv,d,L,P,dtype", [(1, 32, 8, 64, 16400, 200, torch.bfloat16), (1, 40, 40, 64, 16400, 130, torch.float16),
                                                  (1, 56, 8, 64, 16500, 70, torch.bfloat16), (7, 8, 4, 64, 12900, 600, torch.bfloat16),
                                                  (2, 20, 20, 64, 16385, 80, torch.float32)])
def test_every_column_of_every_head_of_a_group(B, Hq, Hkv, d, L, P, dtype):
    tiles, per_xcd = -(-L // 128), B * Hq // 8
    least = -(-256 // tiles)
    assert B * Hq % 8 == 0 and per_xcd // least > 1              # several groups
    g = torch.Generator(device=DEV).manual_seed(L)
    pos = spread(L, P).to(DEV)
    P = pos.numel()
    q = torch.randn(B, Hq, P, d, generator=g, device=DEV).to(dtype)
    k = torch.randn(B, Hkv, L, d, generator=g, device=DEV).to(dtype)
    rows = torch.arange(P, device=DEV)
    per_head = torch.full((B, Hq, L), float("nan"), device=DEV)
    scores = torch.full((B, L), float("nan"), device=DEV)
    zb.zc_probe_saliency(q, k, pos.int(), probe_rows=rows.int(), scores=scores, scores_per_head=per_head)
    for h in range(Hq):
        want = reference(q[:, h:h + 1], k[:, h * Hkv // Hq][:, None], rows, pos)
        rel = ((per_head[:, h].double() - want).abs() / want.clamp(min=1e-30)).max().item()
        assert rel < 3e-5, (h, rel)                              # (the bound of test_scores_of_row_blocks_and_ranges)
    assert torch.allclose(per_head.mean(1), scores, rtol=1e-5, atol=0)


# Few probes, sweep 2 and the mean in one launch (given normalisers; without them two launches may cost less): 1, 15 to 17, 31 and 32 rows (blocks of 16, halves of a head's two by waves of
# their own and by one), fewer heads than waves, one wave more and heads that do not divide by them, columns of less than a
# tile, of whole tiles and one more, 16 a workgroup and (enough of them for more than a round) 32, every probe at one position,
# probes in front of most columns
FEW = [
    (1, 1, 1, 64, 1, torch.float16, lambda L: torch.arange(1)),
    (3, 8, 8, 64, 16, torch.float32, lambda L: torch.arange(1, 16)),
    (2, 8, 2, 128, 17, torch.bfloat16, lambda L: torch.arange(1, 17)),
    (2, 8, 8, 64, 100, torch.float16, lambda L: spread(L, 17)),
    (1, 9, 3, 64, 257, torch.bfloat16, lambda L: spread(L, 31)),
    (1, 16, 16, 128, 33, torch.float32, lambda L: torch.full((16,), 32)),
    (2, 17, 1, 64, 95, torch.float32, lambda L: spread(L, 32)),
    (1, 33, 11, 64, 64, torch.bfloat16, lambda L: torch.arange(5, 37)),
    (12, 24, 8, 128, 700, torch.float32, lambda L: spread(L, 9)),
    (16, 16, 4, 64, 1000, torch.bfloat16, lambda L: torch.arange(480, 496)),
    (9, 8, 4, 128, 1500, torch.float16, lambda L: spread(L, 20)),
]


@pytest.mark.parametrize("external", [False, True])
@pytest.mark.parametrize("case", range(len(FEW)))
def test_scores_of_few_probes_in_one_launch(case, external):
    B, Hq, Hkv, d, L, dtype, probes = FEW[case]
    g = torch.Generator(device=DEV).manual_seed(case)
    pos = probes(L).to(DEV)
    P = pos.numel()
    q = (torch.randn(B, Hq, P + 3, d, generator=g, device=DEV) + 0.25).to(dtype)
    rows = torch.randperm(P + 3, generator=g, device=DEV)[:P]
    k = torch.randn(B, L, Hkv, d, generator=g, device=DEV)                       # a token's heads side by side
    k[..., ::31] *= 15.0
    k = k.to(dtype).transpose(1, 2)
    lse = 40.0 + torch.randn(B, Hq, P, generator=g, device=DEV) if external else None
    want = reference(q, k, rows, pos, lse)
    per_head = torch.full((B, Hq, L), float("nan"), device=DEV)
    got = [zb.zc_probe_saliency(q, k, pos.int(), probe_rows=rows.int(), lse_ext=lse, scores_per_head=ph) for ph in (None, per_head)]
    for s in got:
        rel = ((s.double() - want).abs() / want.clamp(min=1e-30)).max().item()
        assert rel < 3e-5, rel                                                   # (the bound of test_scores_of_row_blocks_and_ranges)
    assert torch.equal(got[0], got[1])
    assert torch.allclose(per_head.mean(1), got[1], rtol=1e-5, atol=0)
    summed = zb.zc_probe_accumulated(q, k, pos.int(), probe_rows=rows.int(), lse_ext=lse)
    seen = (pos[:, None] >= torch.arange(L, device=DEV)[None]).sum(0).clamp(min=1)
    assert torch.allclose(summed / seen, got[0], rtol=1e-5, atol=0)
