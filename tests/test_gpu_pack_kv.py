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
