"""GPU parity of Algorithm 3's re-compression branch taken at its word (explicit probe rows,
re-ranking and re-compression of everything but the newest window) against the oracle's
LiteralStreamingCache: the attention rows zc_decode_probs emits, Eq. 8 on them
(zc_rows_saliency), the de-quantized token buffer (zc_dequantize_cache), the split and the
re-quantized cache, and every decode output, over two windows."""
import numpy as np
import pytest
import torch

from oracle import zipcache_oracle as zo
from paper_2405_14256_amd import binding as zb
from paper_2405_14256_amd import probes
from paper_2405_14256_amd.workloads import WORKLOADS, make_decode_step, make_prefill, scaled, to_f64
from tests.pipeline_check import CODE_COUNTS, assert_code_budgets, check_index_sets, compare_subset, packed_to_chunks

pytestmark = pytest.mark.gpu
DEV = "cuda"


def run_literal(w, interval, windows, extra_steps=3):
    dev = torch.device(DEV)
    lib = zb.load()
    B, Hq, Hkv, d, L = w.B, w.Hq, w.Hkv, w.d, w.L
    bsel = list(range(B))
    steps = windows * interval + extra_steps
    Nmax = L + steps
    fp32 = w.dtype == "fp32"
    atol = 1e-4 if fp32 else 2e-2
    inp = make_prefill(w)
    Qg, Kg, Vg = (inp[n].to(dev) for n in ("Q", "K", "V"))
    pos_np = probes.probe_positions(L, w.probe_ratio, w.seed)
    scores0 = zb.zc_probe_saliency(Qg, Kg, torch.from_numpy(pos_np).to(dev))
    k0 = w.k_salient
    sal, reg = zb.zc_select_salient(scores0, k0)
    m_max = L + (windows - 1) * interval
    k_max = int(np.floor(w.salient_ratio * m_max + 1e-9))
    cap_hi, cap_lo = lib.zc_arena_slots(k_max, 1), lib.zc_arena_slots(m_max - min(k0, k_max), 1)
    def mk(scheme, layout):
        return zb.PackedTensor(B, Hkv, d, cap_hi, cap_lo, w.bits_hi, w.bits_lo, scheme, layout, max_chunks=1, device=DEV)
    caches = [(mk("channel", zb.ZC_LAYOUT_ROW), mk("cst", zb.ZC_LAYOUT_TGROUP)) for _ in range(2)]
    Kp, Vp = caches[0]
    zb.zc_quantize_pack(Kg, sal, reg, Kp)
    zb.zc_quantize_pack(Vg, sal, reg, Vp)
    torch.cuda.synchronize()
    # the token buffers: positions [0, n_packed) are filled by zc_dequantize_cache when a window
    # closes, [n_packed, n) are the full-precision tokens (the decode calls' tail)
    Xk = torch.zeros(B, Hkv, Nmax, d, dtype=w.torch_dtype, device=dev)
    Xv = torch.zeros_like(Xk)
    n_packed = L
    oracle = zo.LiteralStreamingCache(Hkv=Hkv, store_dtype=w.dtype, bits_hi=w.bits_hi, bits_lo=w.bits_lo, interval=interval,
                                      chunk_K=packed_to_chunks(Kp, bsel)[0], chunk_V=packed_to_chunks(Vp, bsel)[0], n_packed=L)
    probe_off = set(probes.decode_probe_offsets(interval, seed=w.seed).tolist())
    n_probe = len(probe_off)
    rows_g = torch.zeros(n_probe, B, Hq, Nmax, dtype=torch.float32, device=dev)
    row_len = []
    rep = {"out": 0.0, "lse": 0.0, "row": 0.0, "score": 0.0, "score_e2e": 0.0, "dequant_mismatch": 0.0}
    totals = {key: 0 for key in CODE_COUNTS}
    prev_sal = set(sal[0].cpu().tolist())
    changed = 0
    for j in range(steps):
        d_in = make_decode_step(w, j)
        n = L + j                                      # position of the new token
        Xk[:, :, n] = d_in["k_new"].to(dev)
        Xv[:, :, n] = d_in["v_new"].to(dev)
        T = n + 1 - n_packed
        qg = d_in["q"].to(dev)
        lse_g = torch.empty(B, Hq, dtype=torch.float32, device=dev)
        out_g = zb.zc_decode_attention(qg, Kp, Vp, Xk[:, :, n_packed:], Xv[:, :, n_packed:], T, lse_out=lse_g)
        is_probe = j < windows * interval and (j % interval) in probe_off
        out_o, lse_o, row_o = oracle.step(to_f64(d_in["q"]), to_f64(d_in["k_new"]), to_f64(d_in["v_new"]), is_probe)
        rep["out"] = max(rep["out"], float(np.abs(to_f64(out_g) - out_o).max()))
        rep["lse"] = max(rep["lse"], float(np.abs(lse_g.cpu().numpy() - lse_o).max()))
        assert rep["out"] <= atol and rep["lse"] <= max(atol, 1e-3), (j, rep)
        if is_probe:
            jp = len(row_len)
            zb.zc_decode_probs(qg, Kp, Xk[:, :, n_packed:], T, n_packed, lse_g, rows_g[jp])
            row_len.append(n + 1)
            got = rows_g[jp, :, :, :n + 1].cpu().numpy().astype(np.float64)
            assert float(rows_g[jp, :, :, n + 1:].abs().sum()) == 0.0           # nothing past the row's tokens
            assert np.allclose(got.sum(-1), 1.0, atol=2e-3 if not fp32 else 1e-5)
            if fp32:
                err = float((np.abs(got - row_o) / np.maximum(row_o, 1e-6 * row_o.max())).max())
                assert err <= 1e-4, (j, err)
            else:
                err = float(np.abs(got - row_o).max())
                assert err <= 2e-3, (j, err)
            rep["row"] = max(rep["row"], err)
        if (j + 1) % interval == 0 and j < windows * interval:
            m = n + 1 - interval
            k = int(np.floor(w.salient_ratio * m + 1e-9))
            rl = torch.tensor(row_len, dtype=torch.int32, device=dev)
            sc_g = zb.zc_rows_saliency(rows_g[:len(row_len)].contiguous(), rl, m)
            # (a) Eq. 8 on the rows the GPU produced; (b) end to end against the oracle's own rows
            sc_dec = zo.rows_saliency([rows_g[i, :, :, :row_len[i]].cpu().numpy().astype(np.float64) for i in range(len(row_len))])[:, :m]
            sg = sc_g.cpu().numpy().astype(np.float64)
            srel = float((np.abs(sg - sc_dec) / np.maximum(sc_dec, 1e-6 * sc_dec.max())).max())
            assert srel <= 1e-5, srel
            Kt_o, Vt_o = oracle.token_matrices()
            sc_o, sal_o, reg_o = oracle.recompress(w.salient_ratio)
            erel = float((np.abs(sg - sc_o) / np.maximum(sc_o, 1e-6 * sc_o.max())).max())
            assert erel <= (1e-4 if fp32 else 3e-3) + 2.0 * rep["lse"], erel
            rep["score"], rep["score_e2e"] = max(rep["score"], srel), max(rep["score_e2e"], erel)
            sal_g, reg_g = zb.zc_select_salient(sc_g, k)
            sal_np, reg_np = sal_g.cpu().numpy(), reg_g.cpu().numpy()
            for b in bsel:
                s_ex, r_ex = zo.select_salient(sc_g[b].cpu().numpy(), k)
                assert np.array_equal(s_ex, sal_np[b]) and np.array_equal(r_ex, reg_np[b])
                if fp32:
                    check_index_sets(sc_o[b], sal_np[b], k, f"window {j // interval} b={b}")
            # the compressed tokens as they now are, at their positions
            zb.zc_dequantize_cache(Kp, Xk)
            zb.zc_dequantize_cache(Vp, Xv)
            torch.cuda.synchronize()
            for Xg, Xo in ((Xk, Kt_o), (Xv, Vt_o)):
                got = to_f64(Xg[:, :, :n + 1])
                ulp = {"fp32": 2.0 ** -22, "fp16": 2.0 ** -10, "bf16": 2.0 ** -7}[w.dtype]
                assert np.all(np.abs(got - Xo) <= ulp * np.abs(Xo) + 1e-30)
                rep["dequant_mismatch"] = max(rep["dequant_mismatch"], float((got != Xo).mean()))
                assert np.array_equal(got[:, :, n_packed:], Xo[:, :, n_packed:])         # the full-precision tokens are untouched
            # (16-bit storage: the kernel's fp32 evaluation and the oracle's fp64 one round to the same
            # stored value except at a rounding boundary; fp32 storage keeps the fp32 evaluation itself)
            assert fp32 or rep["dequant_mismatch"] <= 1e-3
            # re-compression into the other pair of packed tensors
            Kp2, Vp2 = caches[((j + 1) // interval) % 2]
            Kp2.reset(); Vp2.reset()
            zb.zc_quantize_pack(Xk[:, :, :m], sal_g, reg_g, Kp2)
            zb.zc_quantize_pack(Xv[:, :, :m], sal_g, reg_g, Vp2)
            torch.cuda.synchronize()
            ck_g, cv_g = packed_to_chunks(Kp2, bsel)[0], packed_to_chunks(Vp2, bsel)[0]
            ok_ = zo.compress_tensor(to_f64(Xk[:, :, :m]), sal_np, reg_np, w.bits_hi, w.bits_lo, "channel")
            ov_ = zo.compress_tensor(to_f64(Xv[:, :, :m]), sal_np, reg_np, w.bits_hi, w.bits_lo, "cst")
            for name, g_, o_ in (("K.hi", ck_g.hi, ok_.hi), ("K.lo", ck_g.lo, ok_.lo), ("V.hi", cv_g.hi, ov_.hi), ("V.lo", cv_g.lo, ov_.lo)):
                c = compare_subset(g_, o_, f"window {j // interval} {name}")
                print(f"[literal]   {name}: " + " ".join(f"{key}={c[key]}" for key in CODE_COUNTS), flush=True)
                for key in CODE_COUNTS:
                    totals[key] += c[key]
            # the oracle goes on with the cache the GPU holds
            oracle.chunk_K, oracle.chunk_V, oracle.n_packed = ck_g, cv_g, m
            Kp, Vp, n_packed = Kp2, Vp2, m
            rows_g.zero_()
            row_len = []
            now_sal = set(sal_np[0].tolist())
            promoted = len([p for p in now_sal - prev_sal if p < m - interval or j < interval])    # were compressed as regular before
            demoted = len(prev_sal - now_sal)
            changed += promoted + demoted
            prev_sal = now_sal
            print(f"[literal] window {j // interval}: m={m} k={k} row err {rep['row']:.2e} score rel {srel:.1e} / {erel:.1e} end to end; "
                  f"b=0: {promoted} tokens promoted to salient, {demoted} demoted to regular", flush=True)
    # Re-compression quantizes values that sit on the previous quantization grid.  With fp32
    # storage that grid survives exactly, so x / s hits n + 1/2 structurally (a channel whose new
    # range spans an even number of old steps puts every odd old level on a tie), give or take
    # the 1e-7 rounding noise of the stored x_hat; the fp32 kernel rounds the quotient to fp32
    # before it rounds to an integer and so sees a tie where exact arithmetic sees +-1e-7.  Every
    # such element is still one step apart at its rounding boundary (compare_subset); only the
    # budget is wider here.  16-bit storage rounds x_hat off the grid: the usual budget holds.
    rep.update(assert_code_budgets(totals, w.name, level_budget=1e-3 if fp32 else 1e-4))
    print("[literal]", w.name, rep, flush=True)
    assert changed > 0          # the literal reading's signature: tokens change subsets
    return rep


def test_literal_recompression_fp32_two_windows():
    w = scaled(WORKLOADS["tiny"], B=2, Hq=8, Hkv=4, L=150)
    run_literal(w, interval=40, windows=2)


def test_literal_recompression_bf16_grouped_heads_two_windows():
    w = scaled(WORKLOADS["llama3_8b_4k"], B=1, Hq=8, Hkv=2, L=300)
    run_literal(w, interval=100, windows=2)


def test_literal_recompression_fp16_mha():
    w = scaled(WORKLOADS["llama2_13b_4k_b16"], B=2, Hq=4, Hkv=4, L=130)
    run_literal(w, interval=64, windows=2)


def test_decode_probs_over_many_chunks_and_schemes():
    """zc_decode_probs on a chunk-local cache (several chunks, CST keys too): the row sums to one
    and equals the oracle's probabilities in token order."""
    B, Hq, Hkv, d = 2, 8, 2, 64
    g = torch.Generator().manual_seed(21)
    sizes = [150, 70, 33]
    T = 19
    Ltot = sum(sizes) + T
    for dtype, k_scheme in ((torch.float32, "cst"), (torch.bfloat16, "channel"), (torch.float16, "token")):
        K = torch.randn(B, Hkv, Ltot, d, generator=g).to(dtype)
        V = torch.randn(B, Hkv, Ltot, d, generator=g).to(dtype)
        q = torch.randn(B, Hq, d, generator=g).to(dtype)
        lib = zb.load()
        ks = [60, 20, 0]
        cap_hi, cap_lo = lib.zc_arena_slots(sum(ks), 3), lib.zc_arena_slots(sum(sizes) - sum(ks), 3)
        Kp = zb.PackedTensor(B, Hkv, d, cap_hi, cap_lo, 4, 2, k_scheme, zb.ZC_LAYOUT_ROW, max_chunks=3, device=DEV)
        Vp = zb.PackedTensor(B, Hkv, d, cap_hi, cap_lo, 4, 2, "cst", zb.ZC_LAYOUT_TGROUP, max_chunks=3, device=DEV)
        Kd, Vd = K.to(DEV), V.to(DEV)
        n0 = 0
        for n_new, k_new in zip(sizes, ks):
            sal, reg = zb.zc_select_salient(torch.rand(B, n_new, generator=g).to(DEV), k_new)
            zb.zc_quantize_pack(Kd[:, :, n0:n0 + n_new], sal, reg, Kp, pos_offset=n0)
            zb.zc_quantize_pack(Vd[:, :, n0:n0 + n_new], sal, reg, Vp, pos_offset=n0)
            n0 += n_new
        lse = torch.empty(B, Hq, dtype=torch.float32, device=DEV)
        zb.zc_decode_attention(q.to(DEV), Kp, Vp, Kd[:, :, n0:], Vd[:, :, n0:], T, lse_out=lse)
        row = torch.zeros(B, Hq, Ltot + 5, dtype=torch.float32, device=DEV)
        zb.zc_decode_probs(q.to(DEV), Kp, Kd[:, :, n0:], T, n0, lse, row)
        bsel = [0, 1]
        chunks_k, chunks_v = packed_to_chunks(Kp, bsel), packed_to_chunks(Vp, bsel)
        Kc, Vc = zo.cache_matrices(chunks_k, chunks_v, Hkv, K[:, :, n0:].double().numpy(), V[:, :, n0:].double().numpy())
        _, _, probs = zo.decode_attention(q.double().numpy(), Kc, Vc)
        pos = zo.cache_positions(chunks_k, T, n0)
        want = np.zeros((B, Hq, Ltot + 5))
        for b in range(B):
            want[b][:, pos[b]] = probs[b]
        got = row.cpu().numpy().astype(np.float64)
        tol = 1e-4 if dtype == torch.float32 else 2e-3
        if dtype == torch.float32:
            assert (np.abs(got - want) / np.maximum(want, 1e-6 * want.max())).max() <= tol, (dtype, k_scheme)
        else:
            assert np.abs(got - want).max() <= tol, (dtype, k_scheme)
        assert np.all(got[:, :, Ltot:] == 0.0)


@pytest.mark.parametrize("P,B,Hq,N,n_out", [(1, 1, 1, 40, 1), (9, 2, 40, 100, 33), (8, 1, 70, 64, 64), (17, 3, 64, 131, 65), (10, 300, 2, 70, 70),
                                           (3, 12, 1, 300, 257), (15, 128, 1, 260, 256)])
def test_rows_saliency_shapes(P, B, Hq, N, n_out):
    """Columns around the edges of a workgroup's tile (32, 64 and 256 columns), more heads than are
    summed at once, row counts around a batch of rows; cells past a row's length hold NaN."""
    g = torch.Generator().manual_seed(P * 1000 + Hq)
    rows = torch.rand(P, B, Hq, N, generator=g)
    row_len = torch.sort(torch.randint(1, N + 1, (P,), generator=g)).values.to(torch.int32)
    seen = torch.arange(N)[None] < row_len[:, None].long()                       # [P, N]
    rows = torch.where(seen[:, None, None], rows, torch.full((), float("nan")))
    want = torch.where(seen[:, None, None], rows, torch.zeros(())).double().sum(0).mean(1)[:, :n_out]
    cnt = seen.sum(0)[:n_out].double()
    for normalize in (True, False):
        ref = want / cnt.clamp(min=1) if normalize else want
        got = zb.zc_rows_saliency(rows.to(DEV), row_len.to(DEV), n_out, normalize=normalize).cpu().double()
        # P * Hq terms of at most 1 summed in fp32 in two chains
        assert float((got - ref).abs().max()) <= 2.0 ** -24 * (P + Hq) * float(ref.max()) + 1e-12


def test_rows_saliency_of_more_columns_than_a_grid_dimension_counts():
    n = (1 << 28) + 65              # tiles of 64 columns, 1024 threads each: one and a remainder past 2^32 threads
    rows = torch.rand(1, 1, 1, n, device=DEV, generator=torch.Generator(DEV).manual_seed(1))
    got = zb.zc_rows_saliency(rows, torch.tensor([n], dtype=torch.int32, device=DEV), n, scores=torch.zeros(1, n, device=DEV))
    assert torch.equal(got, rows[0, 0])


def _unpacked(p, total, dtype):
    """x_hat of the cache `p` of `total` tokens in token order [B, H, total, d], rounded to dtype:
    fp16 from the exact product of the scales' fp32 product and the level, in one rounding."""
    want = torch.zeros(p.B, total, p.H * p.D, dtype=torch.float64 if dtype == torch.float16 else torch.float32, device=DEV)
    for ci, row in enumerate(p.chunks):
        for which in (0, 1):
            begin, n = row[2 * which:2 * which + 2]
            if n == 0:
                continue
            codes, x = zb.zc_unpack(p, which, ci)
            if dtype == torch.float16:
                scale, level = p.chan_scale[ci, which][:, None], codes.float() - p.chan_zero[ci, which][:, None]
                if p.scheme != "channel":
                    scale = scale * (p.tok_scale_lo if which else p.tok_scale_hi)[:, begin:begin + n, None]
                    level = level - (p.tok_zero_lo if which else p.tok_zero_hi)[:, begin:begin + n, None]
                x = scale.double() * level.double()
            pos = (p.pos_lo if which else p.pos_hi)[:, begin:begin + n].long()
            for b in range(p.B):
                want[b, pos[b]] = x[b]
    if dtype == torch.float16:         # (torch converts float64 to float16 through float32; numpy does not)
        want = torch.from_numpy(want.cpu().numpy().astype(np.float16)).to(DEV)
    return want.to(dtype).view(p.B, total, p.H, p.D).permute(0, 2, 1, 3)


@pytest.mark.parametrize("scheme,layout", [("channel", zb.ZC_LAYOUT_ROW), ("cst", zb.ZC_LAYOUT_TGROUP)])
def test_dequantize_cache_rounds_fp16_once(scheme, layout):
    """Enough 4-bit channels that some products (R / 15 times 3, 5, 6, 9, 10 or 12) lie within an
    fp32 unit of an fp16 midpoint, where a product rounded to fp32 first ends on the other side."""
    B, H, d, L, k = 2, 24, 128, 3000, 2000
    g = torch.Generator().manual_seed(15)
    x = torch.randn(B, H, L, d, generator=g).to(torch.float16).to(DEV)
    p = zb.PackedTensor(B, H, d, 2048, 1024, 4, 2, scheme, layout, max_chunks=1, device=DEV)
    sal, reg = zb.zc_select_salient(torch.rand(B, L, generator=g).to(DEV), k)
    zb.zc_quantize_pack(x, sal, reg, p)
    out = torch.zeros_like(x)
    zb.zc_dequantize_cache(p, out)
    want = _unpacked(p, L, torch.float16)
    assert x.numel() > 10**7 and int((out != want).sum()) == 0


@pytest.mark.parametrize("bits_hi,bits_lo,d,dtype", [(4, 2, 128, torch.bfloat16), (8, 4, 64, torch.float16), (2, 8, 128, torch.float32)])
def test_dequantize_cache_is_the_unpacked_cache_in_token_order(bits_hi, bits_lo, d, dtype):
    """More segments than one launch takes, empty subsets, lengths around a block's edges, both
    layouts; positions past the output are skipped, other rows are untouched."""
    B, H = 2, 3
    sizes = [(64, 64), (1, 0), (0, 1), (33, 65), (16, 15)] + [(5, 9)] * 9
    cap = 64 * 20
    g = torch.Generator().manual_seed(bits_hi)
    total = sum(a + b for a, b in sizes)
    X = torch.randn(B, H, total, d, generator=g).to(dtype).to(DEV)
    for scheme, layout in (("channel", zb.ZC_LAYOUT_ROW), ("cst", zb.ZC_LAYOUT_TGROUP), ("token", zb.ZC_LAYOUT_ROW)):
        p = zb.PackedTensor(B, H, d, cap, cap, bits_hi, bits_lo, scheme, layout, max_chunks=len(sizes), device=DEV)
        n0 = 0
        for k, r in sizes:
            sal, reg = zb.zc_select_salient(torch.rand(B, k + r, generator=g).to(DEV), k)
            zb.zc_quantize_pack(X[:, :, n0:n0 + k + r], sal, reg, p, pos_offset=n0)
            n0 += k + r
        Lout = total - 3
        out = torch.full((B, H, Lout + 2, d), 7.0, dtype=dtype, device=DEV)
        want = _unpacked(p, total, dtype)
        zb.zc_dequantize_cache(p, out[:, :, :Lout])
        assert torch.equal(out[:, :, :Lout], want[:, :, :Lout])
        assert float((out[:, :, Lout:].float() - 7.0).abs().max()) == 0.0


@pytest.mark.parametrize("scheme,layout", [("channel", zb.ZC_LAYOUT_ROW), ("cst", zb.ZC_LAYOUT_TGROUP)])
def test_dequantize_cache_later_chunks_replace_earlier_ones(scheme, layout):
    """Three chunks compressed without a position offset hold the same positions: every row is the
    last chunk's that holds it, each time."""
    B, H, d = 1, 8, 128
    g = torch.Generator().manual_seed(3)
    lens = (6000, 4000, 1000)
    p = zb.PackedTensor(B, H, d, 7040, 7040, 4, 2, scheme, layout, max_chunks=3, device=DEV)
    want = torch.zeros(B, H, lens[0], d, dtype=torch.bfloat16, device=DEV)
    for L in lens:
        x = torch.randn(B, H, L, d, generator=g).to(torch.bfloat16).to(DEV)
        sal, reg = zb.zc_select_salient(torch.rand(B, L, generator=g).to(DEV), L // 2)
        zb.zc_quantize_pack(x, sal, reg, p)
        one = zb.PackedTensor(B, H, d, 3072, 3072, 4, 2, scheme, layout, max_chunks=1, device=DEV)
        zb.zc_quantize_pack(x, sal, reg, one)
        zb.zc_dequantize_cache(one, want)
    for _ in range(5):
        out = torch.zeros_like(want)
        zb.zc_dequantize_cache(p, out)
        assert torch.equal(out, want)


def test_dequantize_cache_of_millions_of_tokens():
    """More threads than one launch counts (8192 channels, 4.3 million tokens): the rows of the last
    positions, which the first and the last tokens hold, arrive."""
    H, d, n = 64, 128, 4_300_032
    p = zb.PackedTensor(1, H, d, n, 0, 2, 2, "channel", zb.ZC_LAYOUT_ROW, max_chunks=1, device=DEV)
    p.chan_scale.fill_(1.0)
    p.chan_zero.fill_(-1.0)
    p.pos_hi[0, :4] = torch.arange(4)
    p.pos_hi[0, -4:] = torch.arange(4, 8)
    p.chunk_table_host[0] = (0, n, 0, 0)
    p.c.n_chunks, p.c.n_hi = 1, n
    out = torch.zeros(1, H, 9, d, dtype=torch.float16, device=DEV)
    zb.zc_dequantize_cache(p, out)
    assert bool((out[:, :, :8] == 1.0).all()) and bool((out[:, :, 8] == 0.0).all())


@pytest.mark.parametrize("B,Hq,Hkv,d,dtype,bits,L,T", [
    (1, 1, 1, 64, torch.float32, (8, 2), 17, 1), (3, 16, 2, 128, torch.bfloat16, (2, 8), 1000, 33),
    (16, 40, 40, 128, torch.float16, (4, 2), 515, 0), (2, 6, 2, 128, torch.float32, (4, 4), 63, 16)])
def test_decode_probs_tiles_and_code_widths(B, Hq, Hkv, d, dtype, bits, L, T):
    """Segments that end inside a 16-slot tile, one to eight query heads per KV head, every code
    width, launches of one and of several tiles a wave, more segments than one launch takes."""
    g = torch.Generator().manual_seed(L)
    lib = zb.load()
    sizes = [L] + [3] * 33
    ks = [L // 3] + [1] * 33
    K = torch.randn(B, Hkv, sum(sizes) + T, d, generator=g).to(dtype).to(DEV)
    q = torch.randn(B, Hq, d, generator=g).to(dtype).to(DEV)
    for scheme in ("channel", "token"):
        p = zb.PackedTensor(B, Hkv, d, lib.zc_arena_slots(sum(ks), 34), lib.zc_arena_slots(sum(sizes) - sum(ks), 34), *bits, scheme,
                            zb.ZC_LAYOUT_ROW, max_chunks=34, device=DEV)
        n0 = 0
        for n, k in zip(sizes, ks):
            sal, reg = zb.zc_select_salient(torch.rand(B, n, generator=g).to(DEV), k)
            zb.zc_quantize_pack(K[:, :, n0:n0 + n], sal, reg, p, pos_offset=n0)
            n0 += n
        Kh = K.float()
        zb.zc_dequantize_cache(p, Kh)
        logits = (q.double().view(B, Hkv, Hq // Hkv, 1, d) * Kh.double()[:, :, None]).sum(-1).view(B, Hq, -1) / d ** 0.5
        lse = torch.logsumexp(logits, -1)
        row = torch.full((B, Hq, n0 + T + 2), -1.0, dtype=torch.float32, device=DEV)
        zb.zc_decode_probs(q, p, K[:, :, n0:] if T else None, T, n0, lse.float(), row)
        want = torch.exp(logits - lse[..., None])
        # a probability is exp of a logit of d fp32 terms: a few units of 2^-24 of the largest
        # partial sum, which the token scale times |code - z| times |q| summed over d bounds by 300
        assert float(((row[:, :, :n0 + T].double() - want) / want).abs().max()) <= 300 * 2.0 ** -23
        assert bool((row[:, :, n0 + T:] == -1.0).all())


# Two tiles at a time (more workgroups than CUs by single tiles): segments that end inside the first and the second tile of a pair, at either's
# end and one after, head widths, groups and code widths, one and several pairs a wave, a tail longer than the segments with several tiles a wave,
# and grids of four and of eight workgroups a head and one without work
@pytest.mark.parametrize("B,Hq,Hkv,d,dtype,bits,sizes,T", [
    (9, 16, 8, 64, torch.bfloat16, (4, 8), [(40, 160), (17, 31), (15, 33)], 5), (16, 40, 40, 128, torch.float32, (4, 2), [(17, 63)], 78), (8, 64, 8, 128, torch.float16, (8, 4), [(48, 97), (16, 64), (65, 32)], 17),
    (5, 9, 9, 64, torch.float32, (2, 4), [(511, 1024)], 32), (16, 24, 12, 64, torch.float16, (4, 4), [(1600, 3201), (20, 80)], 0),
    (16, 24, 12, 128, torch.float16, (4, 2), [(500, 900)], 33), (22, 12, 12, 64, torch.bfloat16, (4, 2), [(53, 20), (134, 31), (27, 18)], 95)])
def test_decode_probs_pairs_of_tiles(B, Hq, Hkv, d, dtype, bits, sizes, T):
    g = torch.Generator().manual_seed(Hq)
    lib = zb.load()
    n_packed = sum(k + n for k, n in sizes)
    assert B * Hkv * sum(-(-k // 16) + -(-n // 16) for k, n in sizes) > 1400
    K = torch.randn(B, Hkv, n_packed + T, d, generator=g).to(dtype).to(DEV)
    q = torch.randn(B, Hq, d, generator=g).to(dtype).to(DEV)
    for scheme in ("channel", "token"):
        p = zb.PackedTensor(B, Hkv, d, lib.zc_arena_slots(sum(k for k, _ in sizes), 3), lib.zc_arena_slots(sum(n for _, n in sizes), 3), *bits, scheme,
                            zb.ZC_LAYOUT_ROW, max_chunks=3, device=DEV)
        n0 = 0
        for k, n in sizes:
            sal, reg = zb.zc_select_salient(torch.rand(B, k + n, generator=g).to(DEV), k)
            zb.zc_quantize_pack(K[:, :, n0:n0 + k + n], sal, reg, p, pos_offset=n0)
            n0 += k + n
        Kh = K.float()
        zb.zc_dequantize_cache(p, Kh)
        logits = torch.cat([torch.matmul(q.double().view(B, Hkv, Hq // Hkv, d), k.double().transpose(-1, -2).contiguous()).view(B, Hq, -1)
                            for k in Kh.split(512, 2)], -1) / d ** 0.5
        lse = torch.logsumexp(logits, -1)
        row = torch.full((B, Hq, n0 + T + 2), -1.0, dtype=torch.float32, device=DEV)
        zb.zc_decode_probs(q, p, K[:, :, n0:] if T else None, T, n0, lse.float(), row)
        want = torch.exp(logits - lse[..., None])
        # (the bound of test_decode_probs_tiles_and_code_widths; a chunk of fifteen tokens and more has no channel of a narrow range)
        assert float(((row[:, :, :n0 + T].double() - want) / want).abs().max()) <= 300 * 2.0 ** -23
        assert bool((row[:, :, n0 + T:] == -1.0).all())


@pytest.mark.parametrize("dtype", [torch.float32, torch.float16, torch.bfloat16])
@pytest.mark.parametrize("bits", [(8, 8), (8, 4)])
def test_decode_probs_error_against_64_bits(bits, dtype):
    """The root mean square error of the probabilities over wide codes and outlier key channels:
    the query is held to 22 bits and its products with the centred codes are summed in fp32, so a
    logit (and with it, relatively, a probability) is off by a fraction of 2^-21 of the logits' spread
    (measured 0.2 to 0.35 of 2^-20; 0.5 to 2.3 with codes that are not centred)."""
    B, Hkv, G, d, L, k = 2, 8, 4, 128, 1501, 450
    g = torch.Generator().manual_seed(bits[1])
    K = torch.randn(B, Hkv, L, d, generator=g)
    K[..., ::21] *= 15.0
    K = K.to(dtype).to(DEV)
    q = (torch.randn(B, Hkv * G, d, generator=g) + 0.25).to(dtype).to(DEV)
    sal, reg = zb.zc_select_salient(torch.rand(B, L, generator=g).to(DEV), k)
    for scheme in ("channel", "token", "cst"):
        p = zb.PackedTensor(B, Hkv, d, 512, 1088, *bits, scheme, zb.ZC_LAYOUT_ROW, max_chunks=1, device=DEV)
        zb.zc_quantize_pack(K, sal, reg, p)
        Kh = torch.empty(B, Hkv, L, d, dtype=torch.float32, device=DEV)
        zb.zc_dequantize_cache(p, Kh)
        logits = (q.double().view(B, Hkv, G, 1, d) * Kh.double()[:, :, None]).sum(-1).view(B, Hkv * G, L) / d ** 0.5
        lse = torch.logsumexp(logits, -1).float()
        row = torch.empty(B, Hkv * G, L, dtype=torch.float32, device=DEV)
        zb.zc_decode_probs(q, p, None, 0, L, lse, row)
        want = torch.exp(logits - lse.double()[..., None])
        err = float(((row.double() - want) / want).square().mean().sqrt())
        assert err <= 2.0 ** -21 * float(logits.square().mean().sqrt()), (scheme, err, float(logits.square().mean().sqrt()) * 2.0 ** -20)


@pytest.mark.parametrize("scheme,layout", [("channel", zb.ZC_LAYOUT_ROW), ("token", zb.ZC_LAYOUT_ROW), ("cst", zb.ZC_LAYOUT_TGROUP)])
def test_parameter_arrays_aligned_to_their_elements_only(scheme, layout):
    """Positions, token and channel parameters one element past a 16-byte boundary, which the
    validation admits: the same rows and probabilities."""
    B, H, d, L, k = 2, 3, 128, 150, 50
    g = torch.Generator().manual_seed(8)
    x = torch.randn(B, H, L, d, generator=g).to(torch.bfloat16).to(DEV)
    p = zb.PackedTensor(B, H, d, 64, 128, 4, 2, scheme, layout, max_chunks=1, device=DEV)
    sal, reg = zb.zc_select_salient(torch.rand(B, L, generator=g).to(DEV), k)
    zb.zc_quantize_pack(x, sal, reg, p)
    q = torch.randn(B, 2 * H, d, generator=g).to(torch.bfloat16).to(DEV)
    lse = torch.zeros(B, 2 * H, device=DEV)

    def results():
        out = [torch.zeros_like(x)]
        zb.zc_dequantize_cache(p, out[0])
        if layout == zb.ZC_LAYOUT_ROW:
            out.append(torch.zeros(B, 2 * H, L, device=DEV))
            zb.zc_decode_probs(q, p, None, 0, L, lse, out[1])
        return out
    want, keep = results(), []
    for name in ("tok_scale_hi", "tok_zero_hi", "tok_scale_lo", "tok_zero_lo", "pos_hi", "pos_lo", "chan_scale", "chan_zero"):
        t = getattr(p, name)
        moved = torch.empty(t.numel() + 1, dtype=t.dtype, device=DEV)[1:]
        moved.copy_(t.flatten())
        keep.append(moved)
        setattr(p.c, name, moved.data_ptr())
        assert moved.data_ptr() % 16 == 4
    for a, b in zip(want, results()):
        assert torch.equal(a, b)
