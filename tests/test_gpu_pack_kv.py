"""The packing launch of channelwise ROW keys and channel-separable TGROUP values at the edges of
its pieces (4 keys a thread, word groups of 4, 8 and 16 values, blocks of 4 groups, rows of less
than a wave, of exactly and just over a workgroup), for inputs stored token-major, against the
oracle.  Token rows of both subsets at every size; the budget for codes is that of the randomized
shapes (quotients next to a rounding boundary in fp32)."""
import pytest
import torch

from oracle import zipcache_oracle as zo

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("H,D", [(1, 64), (5, 64), (9, 64), (16, 128), (17, 128)])
@pytest.mark.parametrize("bits_hi,bits_lo", [(4, 2), (8, 4), (2, 8)])
def test_pack_edges(H, D, bits_hi, bits_lo):
    from paper_2405_14256_amd import binding as zb
    from tests.pipeline_check import compare_subset, packed_to_chunks
    B, total, mism = 2, 0, 0
    sizes = [(1, 0), (3, 1), (4, 5), (8, 9), (17, 15), (16, 63), (65, 64), (33, 129)]
    for i, (k, n) in enumerate(sizes):
        L, dtype = k + n, (torch.bfloat16, torch.float16, torch.float32)[i % 3]
        g = torch.Generator().manual_seed(100 * i + H)
        X = (3 * torch.randn(B, L, H, D, generator=g)).to(dtype).to("cuda").permute(0, 2, 1, 3)        # [B, H, L, D], a token's heads adjacent
        Y = torch.randn(B, L, H, D, generator=g).to(dtype).to("cuda").permute(0, 2, 1, 3)
        perm = torch.stack([torch.randperm(L, generator=g) for _ in range(B)])
        sal, reg = (t.sort(dim=1).values.to(torch.int32) for t in (perm[:, :k], perm[:, k:]))
        cap = zb.load().zc_arena_slots(L, 1)
        pack = [zb.PackedTensor(B, H, D, cap, cap, bits_hi, bits_lo, s, lay, max_chunks=1, device="cuda")
                for s, lay in (("channel", zb.ZC_LAYOUT_ROW), ("cst", zb.ZC_LAYOUT_TGROUP))]
        zb.zc_quantize_pack_kv(X, Y, sal.cuda(), reg.cuda(), *pack)
        torch.cuda.synchronize()
        for P, T, scheme in ((pack[0], X, "channel"), (pack[1], Y, "cst")):
            got = packed_to_chunks(P, list(range(B)))[0]
            ref = zo.compress_tensor(T.cpu().double().numpy(), sal.numpy(), reg.numpy(), bits_hi, bits_lo, scheme)
            for a, b, which in ((got.hi, ref.hi, "hi"), (got.lo, ref.lo, "lo")):
                r = compare_subset(a, b, f"{scheme} {k} {n} {dtype} {which}")
                total += r["n_codes"]
                mism += r["n_mismatch"]
            assert torch.equal(P.pos_hi[:, :k].cpu(), sal) and torch.equal(P.pos_lo[:, :n].cpu(), reg)
    assert mism <= 1e-4 * total, (mism, total)


@pytest.mark.parametrize("H,bits_hi,bits_lo", [(17, 4, 2), (40, 8, 4)])
def test_wide_rows_whose_zero_points_leave_the_rounding_range(H, bits_hi, bits_lo):
    """Rows of ones in which one channel is 2^-24 less: zero points of 10^8, beyond what the sums with
    1.5 * 2^23 hold.  The codes follow from the stored z as clamp(rint(x / s) + z) in fp32; the
    quotients are exact (s is a power of two over 2^bits - 1), so there is no tolerance."""
    import numpy as np
    from paper_2405_14256_amd import binding as zb
    from tests import packfmt
    D, L, k, cap = 128, 75, 33, 64
    X = torch.ones(1, H, L, D)
    rows = [0, 7, 32, 33, 74]
    for t in rows:
        X[0, t % H, t, 5] = 1.0 - 2.0 ** -24
    sal, reg = torch.arange(0, k, dtype=torch.int32)[None], torch.arange(k, L, dtype=torch.int32)[None]
    P = zb.PackedTensor(1, H, D, cap, cap, bits_hi, bits_lo, "cst", zb.ZC_LAYOUT_TGROUP, max_chunks=1, device="cuda")
    zb.zc_quantize_pack(X.cuda(), sal.cuda(), reg.cuda(), P)
    torch.cuda.synchronize()
    for idx, bits, codes, z in ((sal[0], bits_hi, P.codes_hi, P.tok_zero_hi), (reg[0], bits_lo, P.codes_lo, P.tok_zero_lo)):
        got = packfmt.decode_tgroup(codes.cpu().numpy(), 1, H, D, cap, bits)[0]           # [H, cap, D]
        z = z.cpu().numpy()[0]
        qmax = np.float32(2 ** bits - 1)
        for j, t in enumerate(idx.tolist()):
            inv_s = qmax * np.float32(2.0 ** 24) if t in rows else np.float32(1.0)
            assert (abs(z[j]) > 2.0 ** 21) == (t in rows)
            want = np.clip(np.rint(X[0, :, t].numpy() * inv_s) + z[j], 0, qmax)
            assert np.array_equal(got[:, j], want), (bits, t)
