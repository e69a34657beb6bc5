"""GPU parity of zc_prefill_attention (Algorithm 2's attention line) against the oracle,
and of the probe stage fed with its row normalisers."""
import numpy as np
import pytest
import torch

from oracle import zipcache_oracle as zo
from paper_2405_14256_amd import binding as zb
from paper_2405_14256_amd import probes
from paper_2405_14256_amd.workloads import WORKLOADS, make_prefill, scaled

pytestmark = pytest.mark.gpu
DEV = "cuda"


def _check_heads(w, inp, out, lse, heads, b=0, sm_scale=None, what=""):
    """Output and log-normaliser of the given query heads of batch element b, all rows."""
    G = w.Hq // w.Hkv
    atol = 1e-4 if w.dtype == "fp32" else 2e-2
    ltol = 1e-4 if w.dtype == "fp32" else 1e-3
    worst = [0.0, 0.0]
    for h in heads:
        Q = inp["Q"][b:b + 1, h:h + 1].double().numpy()
        K = inp["K"][b:b + 1, h // G:h // G + 1].double().numpy()
        V = inp["V"][b:b + 1, h // G:h // G + 1].double().numpy()
        O_o, lse_o = zo.prefill_attention(Q, K, V, sm_scale)
        e = np.abs(out[b, h].double().cpu().numpy() - O_o[0, 0]).max()
        le = np.abs(lse[b, h].double().cpu().numpy() - lse_o[0, 0]).max()
        worst = [max(worst[0], e), max(worst[1], le)]
        assert e <= atol, (what, b, h, e)
        assert le <= ltol, (what, b, h, le)
    print(f"[prefill] {what or w.name}: heads {list(heads)} of b={b}: max |out err| {worst[0]:.3e}, max |lse err| {worst[1]:.3e}", flush=True)


def test_prefill_tiny_fp32_every_head():
    w = WORKLOADS["tiny"]
    inp = make_prefill(w)
    out, lse, _ = zb.zc_prefill_attention(inp["Q"].to(DEV), inp["K"].to(DEV), inp["V"].to(DEV))
    _check_heads(w, inp, out, lse, range(w.Hq))


def test_prefill_llama3_8b_4k_sampled_heads():
    w = WORKLOADS["llama3_8b_4k"]
    inp = make_prefill(w)
    out, lse, _ = zb.zc_prefill_attention(inp["Q"].to(DEV), inp["K"].to(DEV), inp["V"].to(DEV))
    _check_heads(w, inp, out, lse, [0, 13, 31])


@pytest.mark.parametrize("name,kw,heads", [
    ("llama3_8b_32k", dict(L=3000, needles=8), [0, 5, 31]),                 # long-context law, ragged against every tile
    ("llama2_13b_4k_b16", dict(B=2, Hq=4, Hkv=4, L=701), [0, 3]),           # fp16, one query head per KV head
    ("mistral_7b_8k_b8", dict(B=2, Hq=8, Hkv=2, L=129), [1, 6]),            # one row past a row block
    ("tiny", dict(L=63, Hq=4, Hkv=2), [0, 3]),                              # fp32, grouped heads, less than one tile
    ("tiny", dict(L=1), [0]),
    ("llama3_8b_4k", dict(L=520, dtype="fp32", Hq=4, Hkv=2), [0, 3]),       # fp32 at head_dim 128
    ("llama3_8b_4k", dict(L=300, dtype="fp16", Hq=2, Hkv=1), [0, 1]),
])
def test_prefill_shapes_and_types(name, kw, heads):
    w = scaled(WORKLOADS[name], **kw)
    inp = make_prefill(w)
    out, lse, _ = zb.zc_prefill_attention(inp["Q"].to(DEV), inp["K"].to(DEV), inp["V"].to(DEV))
    for b in sorted({0, w.B - 1}):
        _check_heads(w, inp, out, lse, heads, b=b, what=f"{name} {kw}")


def test_prefill_strided_views_and_scale_override():
    """Inputs and output as strided views of larger buffers (a fused QKV projection's layout),
    and a softmax scale of the caller's."""
    w = scaled(WORKLOADS["llama3_8b_4k"], L=333, Hq=8, Hkv=2, B=2)
    inp = make_prefill(w)
    big = torch.zeros(w.B, w.L, (w.Hq + 2 * w.Hkv) * w.d + 64, dtype=w.torch_dtype, device=DEV)

    def view(h0, H):
        return big[:, :, h0 * w.d:(h0 + H) * w.d].view(w.B, w.L, H, w.d).permute(0, 2, 1, 3)
    Qv, Kv, Vv = view(0, w.Hq), view(w.Hq, w.Hkv), view(w.Hq + w.Hkv, w.Hkv)
    Qv.copy_(inp["Q"]); Kv.copy_(inp["K"]); Vv.copy_(inp["V"])
    obuf = torch.zeros(w.B, w.L, w.Hq * w.d + 32, dtype=w.torch_dtype, device=DEV)
    Ov = obuf[:, :, :w.Hq * w.d].view(w.B, w.L, w.Hq, w.d).permute(0, 2, 1, 3)
    out, lse, _ = zb.zc_prefill_attention(Qv, Kv, Vv, sm_scale=0.05, out=Ov)
    _check_heads(w, inp, out, lse, [0, 7], b=1, sm_scale=0.05, what="strided views")
    assert float(obuf[:, :, w.Hq * w.d:].abs().sum()) == 0.0              # nothing written past the rows


def test_probe_saliency_from_the_prefill_normalisers():
    """The probe stage given the prefill pass's log-normalisers (one sweep instead of two): the
    scores must be those of the two-sweep path and of the oracle, and select the same tokens."""
    w = scaled(WORKLOADS["llama3_8b_4k"], L=2500)
    inp = make_prefill(w)
    Q, K, V = (inp[n].to(DEV) for n in ("Q", "K", "V"))
    pos_np = probes.probe_positions(w.L, w.probe_ratio, w.seed)
    pos = torch.from_numpy(pos_np).to(DEV)
    _, lse, lse_p = zb.zc_prefill_attention(Q, K, V, probe_pos=pos)
    assert torch.equal(lse_p, lse[:, :, pos.long()])
    one = zb.zc_probe_saliency(Q, K, pos, lse_ext=lse_p)
    two = zb.zc_probe_saliency(Q, K, pos)
    ref, _ = zo.saliency_scores(inp["Q"].double().numpy(), inp["K"].double().numpy(), pos_np)
    got = one.cpu().double().numpy()
    rel = np.abs(got - ref) / np.maximum(ref, 1e-6 * ref.max())
    assert rel.max() <= 1e-4, rel.max()
    assert (one - two).abs().max() <= 1e-4 * two.abs().max()
    s1, _ = zb.zc_select_salient(one, w.k_salient)
    from tests.pipeline_check import check_index_sets
    check_index_sets(ref[0], s1[0].cpu().numpy(), w.k_salient, "split on one-sweep scores")


@pytest.mark.parametrize("dtype", ["bf16", "fp16"])
@pytest.mark.parametrize("B,Hq,Hkv,d,L,rise", [
    (1, 2, 1, 128, 1, 0.0), (1, 3, 3, 64, 31, 0.0), (1, 4, 2, 128, 33, 0.0), (1, 2, 2, 64, 64, 0.0), (1, 8, 2, 128, 65, 0.0),
    (2, 12, 4, 128, 257, 0.0),              # heads that do not divide over the XCDs
    (8, 64, 64, 64, 97, 0.0),               # fewer rows than waves
    (4, 32, 8, 128, 1025, 0.0), (4, 32, 4, 64, 1057, 0.0),      # many tiles, one row past a block and one wave more
    (1, 4, 2, 128, 700, 40.0), (4, 32, 8, 128, 1025, 40.0),     # logits that climb by 2^40 and more: the reference of a row moves
])
def test_prefill_tiles_and_reference(dtype, B, Hq, Hkv, d, L, rise):
    """Edges of row blocks, waves and key halves, and rows whose largest logit keeps growing."""
    dt = {"bf16": torch.bfloat16, "fp16": torch.float16}[dtype]
    g = torch.Generator().manual_seed(L + d + Hq)
    Q = torch.randn(B, Hq, L, d, generator=g)
    K = torch.randn(B, Hkv, L, d, generator=g)
    V = torch.randn(B, Hkv, L, d, generator=g)
    if rise:
        Q[..., 0] = 4.0
        K[..., 0] = torch.linspace(0, rise * d ** 0.5 / 4.0, L)
    Q, K, V = Q.to(dt), K.to(dt), V.to(dt)
    out, lse, _ = zb.zc_prefill_attention(Q.to(DEV), K.to(DEV), V.to(DEV))
    G = Hq // Hkv
    # each weight is rounded once to the type (unit u), and so is the result: both are at most u / 2 of max |V|
    u = 2.0 ** (-8 if dtype == "bf16" else -11)
    for b, h in {(0, 0), (B - 1, Hq - 1), (B // 2, Hq // 2)}:
        O_o, lse_o = zo.prefill_attention(*(t.double().numpy() for t in (Q[b:b + 1, h:h + 1], K[b:b + 1, h // G:h // G + 1], V[b:b + 1, h // G:h // G + 1])))
        vmax = float(V[b, h // G].abs().max())
        assert np.abs(out[b, h].double().cpu().numpy() - O_o[0, 0]).max() <= u * vmax + 1e-5 * vmax
        # fp32 sums of d products: a logit is off by about d 2^-24 of the sum of magnitudes
        assert np.abs(lse[b, h].double().cpu().numpy() - lse_o[0, 0]).max() <= 1e-4 + 2e-5 * rise


@pytest.mark.parametrize("B,Hq,Hkv,d,L", [
    (1, 4, 2, 64, 31), (1, 3, 1, 128, 33), (2, 12, 4, 64, 129), (1, 8, 2, 128, 161),    # a row block's keys over four waves: one to six blocks of them
    (5, 32, 8, 64, 640), (5, 32, 8, 128, 609),                                          # over two
    (5, 32, 8, 64, 865), (5, 32, 4, 128, 833)])                                         # not split
def test_prefill_fp32_key_splits(B, Hq, Hkv, d, L):
    g = torch.Generator().manual_seed(L + d)
    Q, K, V = (torch.randn(B, H, L, d, generator=g) for H in (Hq, Hkv, Hkv))
    K[..., 0] += torch.linspace(0, 20, L)                # the largest logits of a row are not all in one wave's blocks
    out, lse, _ = zb.zc_prefill_attention(Q.to(DEV), K.to(DEV), V.to(DEV))
    G = Hq // Hkv
    for b, h in {(0, 0), (B - 1, Hq - 1)}:
        O_o, lse_o = zo.prefill_attention(*(t.double().numpy() for t in (Q[b:b + 1, h:h + 1], K[b:b + 1, h // G:h // G + 1], V[b:b + 1, h // G:h // G + 1])))
        # a logit of magnitude 2^5 is off by a few of its units 2^-19, a weight by as much relatively, |V| stays below 2^3
        assert np.abs(out[b, h].double().cpu().numpy() - O_o[0, 0]).max() <= 1e-4
        assert np.abs(lse[b, h].double().cpu().numpy() - lse_o[0, 0]).max() <= 1e-4


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float16])
def test_prefill_long_rows(dtype):
    """Eight waves a workgroup (rows of 128 channels from 16384 on): the first and last rows and those
    around a block's edge, against float64; one row past a block."""
    Hq, Hkv, d, L = 8, 2, 128, 16385
    g = torch.Generator().manual_seed(5)
    Q, K, V = (torch.randn(1, H, L, d, generator=g).to(dtype).to(DEV) for H in (Hq, Hkv, Hkv))
    out, lse, _ = zb.zc_prefill_attention(Q, K, V)
    u = 2.0 ** (-8 if dtype == torch.bfloat16 else -11)
    rows = torch.cat([torch.arange(0, 70), torch.arange(8180, 8200), torch.arange(L - 300, L)]).to(DEV)
    for h in (0, 5):
        k, v = K[0, h // 4].double(), V[0, h // 4].double()
        logits = Q[0, h, rows].double() @ k.T / d ** 0.5
        logits.masked_fill_(torch.arange(L, device=DEV)[None] > rows[:, None], float("-inf"))
        want_lse = torch.logsumexp(logits, -1)
        want = torch.exp(logits - want_lse[:, None]) @ v
        vmax = float(v.abs().max())
        # each weight is rounded once to the type (unit u), and so is the result: both are at most u / 2 of max |V|
        assert float((out[0, h, rows].double() - want).abs().max()) <= u * vmax + 1e-5 * vmax
        assert float((lse[0, h, rows].double() - want_lse).abs().max()) <= 1e-4


# Waves that share a row's keys, two and four of them: less than a block of 32 keys, a block and one more, a wave without
# keys, tiles of 64 and of 128 keys whole and one more, rows past the end of a workgroup's second block, several tiles, token-major
# tensors, more workgroups than places, key blocks in which every logit is -inf.  (The first line's first three and the last line's take one wave a row: either
# side of where the rule draws its line; 640 heads of up to 64 rows two; (4, 8, 2, 128, 301) to (2, 16, 16, 64, 1201) and the last line but one two, the others four)
SPLIT = [(1, 3, 1, 64, 31), (2, 4, 4, 64, 33), (1, 8, 2, 128, 64), (3, 4, 1, 128, 65), (1, 5, 5, 64, 97), (1, 8, 8, 64, 128), (2, 8, 4, 128, 129),
         (1, 8, 2, 64, 257), (1, 16, 4, 64, 700), (1, 2, 1, 128, 1500), (4, 8, 2, 128, 301), (2, 24, 8, 128, 481), (1, 32, 8, 128, 840),
         (2, 16, 16, 64, 1201), (1, 8, 8, 64, 3003),
         (20, 32, 8, 64, 31), (20, 32, 32, 64, 33), (20, 32, 4, 64, 64), (1, 4, 4, 128, 96), (1, 4, 4, 128, 97),
         (12, 8, 4, 128, 97), (4, 32, 8, 128, 128), (8, 8, 8, 128, 129),
         (16, 32, 8, 64, 32), (1, 8, 8, 128, 32), (4, 32, 8, 64, 129), (40, 32, 8, 128, 65)]


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float16])
@pytest.mark.parametrize("case", SPLIT)
def test_rows_whose_keys_waves_share(case, dtype):
    B, Hq, Hkv, d, L = case
    g = torch.Generator(device=DEV).manual_seed(L)
    Q, K, V = (torch.randn(B, L, h, d, generator=g, device=DEV).to(dtype).transpose(1, 2) for h in (Hq, Hkv, Hkv))
    Q = Q.clone(memory_format=torch.preserve_format)
    Q[..., 1] = 1.0
    if L > 300:
        K[:, :, 64:96, 1] = K[:, :, 160:224, 1] = -float("inf")
    pos = torch.randint(0, L, (min(L, 40),), generator=g, device=DEV).sort().values.int()
    out, lse, lse_p = zb.zc_prefill_attention(Q, K, V, probe_pos=pos)
    assert torch.equal(lse_p, lse[:, :, pos.long()])
    # a weight and the result are rounded to the type (8 and 11 significant bits: by 2^-8 and 2^-11 of their size; weights in fp16
    # from 2^-14 on down by 2^-25), a logit, of up to 2^6, is an fp32 sum of 128 products: 2^-18 at most
    u, low = (2.0 ** -8, 0.0) if dtype == torch.bfloat16 else (2.0 ** -11, 2.0 ** -25)
    hidden = torch.ones(L, L, dtype=torch.bool, device=DEV).triu(1)
    for b in range(B):
        for h in range(Hq):
            k, v = K[b, h * Hkv // Hq].double(), V[b, h * Hkv // Hq].double()
            x = (Q[b, h].double() @ k.T / d ** 0.5).masked_fill(hidden, -float("inf"))
            p = torch.softmax(x, -1)
            want, size = p @ v, p @ v.abs()
            bound = (1.01 * u + 2.0 ** -17) * (size + want.abs()) + low * v.abs().sum(0)
            assert bool(((out[b, h].double() - want).abs() <= bound).all()), (b, h)
            assert (lse[b, h].double() - torch.logsumexp(x, -1)).abs().max().item() <= 1e-4


# The first 40 keys of every row, more than its first block, have logits of -inf: a reference that starts there is still finite.  One case
# for each kernel: fp32 by 16 rows, by 32 rows of four, two and one wave, 16-bit types by four, two and one wave a row and by 256 rows
NO_LOGITS = [(1, 8, 64, 100, torch.float32), (1, 24, 64, 700, torch.float32), (4, 32, 64, 800, torch.float32), (5, 32, 128, 870, torch.float32),
             (1, 8, 64, 300, torch.bfloat16), (1, 16, 128, 1500, torch.float16), (4, 32, 128, 1500, torch.bfloat16), (8, 32, 64, 700, torch.float16),
             (1, 8, 128, 16384, torch.float16)]


@pytest.mark.parametrize("case", NO_LOGITS)
def test_rows_whose_first_logits_are_minus_infinity(case):
    B, H, d, L, dtype = case
    g = torch.Generator(device=DEV).manual_seed(L)
    Q, K, V = (torch.randn(B, H, L, d, generator=g, device=DEV).to(dtype) for _ in range(3))
    Q[..., 1] = 1.0
    K[:, :, :40, 1] = -float("inf")
    out, lse, _ = zb.zc_prefill_attention(Q, K, V)
    rows = torch.tensor([40, 41, 63, 64, 95, 96, L // 2, L - 1], device=DEV)
    hidden = torch.arange(L, device=DEV)[None] > rows[:, None]
    u = {torch.float32: 2.0 ** -20, torch.bfloat16: 2.0 ** -8, torch.float16: 2.0 ** -10}[dtype]
    for b, h in ((0, 0), (B - 1, H - 1)):
        x = (Q[b, h, rows].double() @ K[b, h].double().T / d ** 0.5).masked_fill(hidden, -float("inf"))
        v = V[b, h].double()
        p = torch.softmax(x, -1)
        # (the weights and the result are rounded to the type; fp32: a logit's and the weights' sums, 2^-20 of their size)
        assert bool(((out[b, h, rows].double() - p @ v).abs() <= 2 * u * (p @ v.abs()) + 1e-6).all()), (b, h)
        assert (lse[b, h, rows].double() - torch.logsumexp(x, -1)).abs().max().item() <= 1e-4
    assert bool(out[:, :, 40:].isfinite().all()) and bool(lse[:, :, 40:].isfinite().all())
