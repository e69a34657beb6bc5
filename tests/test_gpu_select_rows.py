"""zc_select_salient on rows around the sizes at which its workgroup changes, against the oracle:
exact index lists and mask.  Rows that need one digit pass, two (hundreds of keys that share the
first digit), all of them (more equal keys than the bisection holds, straddling the k-th place),
and none (one value)."""
import numpy as np
import pytest
import torch

from oracle import zipcache_oracle as zo

pytestmark = pytest.mark.gpu


def _row(kind, n, rng):
    if kind == "spread":
        return np.exp(rng.standard_normal(n)).astype(np.float32) / n
    if kind == "one_digit":                 # neighbours in the last bits of one float, one outlier
        x = (np.float32(1.0).view(np.uint32) + rng.integers(0, 700, n).astype(np.uint32)).view(np.float32)
        x[n // 2] = 1e9
        return x
    if kind == "ties":
        return np.where(rng.random(n) < 0.8, np.float32(0.25), rng.standard_normal(n).astype(np.float32))
    return np.full(n, -0.5, np.float32)


@pytest.mark.parametrize("L", [2, 63, 256, 257, 1024, 1025, 2048, 2049, 4096, 4097, 8192, 8193, 16384, 16385])
def test_select_rows(L):
    from paper_2405_14256_amd import binding as zb
    rng = np.random.default_rng(L)
    x = np.stack([_row(kind, L, rng) for kind in ("spread", "one_digit", "ties", "const", "spread")])
    for k in sorted({0, 1, L // 3, L // 2, L - 1, L}):
        mask = torch.full((x.shape[0], L), 7, dtype=torch.uint8, device="cuda")
        sal, reg = zb.zc_select_salient(torch.from_numpy(x).cuda(), k, mask=mask)
        for b in range(x.shape[0]):
            s_o, r_o = zo.select_salient(x[b].astype(np.float64), k)
            assert np.array_equal(sal[b].cpu().numpy(), s_o) and np.array_equal(reg[b].cpu().numpy(), r_o), (L, k, b)
            m = np.zeros(L, np.uint8)
            m[s_o] = 1
            assert np.array_equal(mask[b].cpu().numpy(), m), (L, k, b)


def _check(x, k):
    from paper_2405_14256_amd import binding as zb
    sal, reg = zb.zc_select_salient(x, k)
    first = torch.sort(x, dim=1, descending=True, stable=True).indices            # equal scores: lower index first
    assert torch.equal(sal.long(), first[:, :k].sort(dim=1).values) and torch.equal(reg.long(), first[:, k:].sort(dim=1).values)


@pytest.mark.parametrize("L", [700, 1500, 3001, 5000, 12001, 16383])
def test_select_rows_of_few_values(L):
    """Rows in which most keys share a digit: one or two values, values of either sign (no bit is shared:
    pads look like keys of the lowest digit), close values beside one far away, and almost only -inf."""
    g = torch.Generator(device="cuda").manual_seed(L)
    u, v = torch.rand(2, L, generator=g, device="cuda"), torch.randn(L, generator=g, device="cuda")
    lowest = torch.finfo(torch.float32).min
    rows = [torch.where(u[0] < 0.9, torch.zeros_like(v), v.exp()), torch.where(u[0] < 0.45, torch.zeros_like(v), torch.where(u[0] < 0.9, torch.ones_like(v), v)),
            torch.where(u[0] < 0.9, -torch.ones_like(v), torch.ones_like(v)), v, 1.0 + 1e-5 * u[1], torch.where(u[0] < 0.97, torch.full_like(v, float("-inf")), v),
            torch.where(u[0] < 0.5, torch.full_like(v, float("-inf")), torch.full_like(v, lowest)), torch.where(u[0] < 0.97, torch.full_like(v, float("inf")), v)]
    rows[4][L // 2] = 1e9
    x = torch.stack(rows)
    for k in (1, 37, L // 20, L // 3, L // 2, L - L // 20, L - 1):
        _check(x, k)


@pytest.mark.parametrize("B,L", [(257, 8193), (257, 15616), (257, 15617), (769, 4097), (769, 8192), (256, 9000)])
def test_select_many_rows(B, L):
    g = torch.Generator(device="cuda").manual_seed(B)
    x = torch.randn(B, L, generator=g, device="cuda").exp()
    x[::3] = (x[::3] * 8).floor()
    _check(x, L // 3)


@pytest.mark.parametrize("B,L", [(32, 2049), (33, 2049), (32, 4096), (33, 4095), (32, 4097), (33, 8192), (32, 8193), (33, 16384), (32, 16384),
                                 (1, 16385), (2, 16640), (4, 21001), (32, 30000), (33, 30000), (3, 34816), (33, 34815), (2, 34817)])
def test_select_rows_shared_by_workgroups(B, L):
    """Rows that eight workgroups share (up to 32 of them) and that one takes: spread scores, few values (the k-th place inside
    thousands of equal ones, over many pieces), one value, and a row of -inf, salient counts down to none of a piece and all of it."""
    from paper_2405_14256_amd import binding as zb
    g = torch.Generator(device="cuda").manual_seed(B + L)
    x = torch.randn(B, L, generator=g, device="cuda").exp()
    if B > 1:
        x[1] = (x[1] * 2).floor()
        x[B - 1] = float("-inf")
    if B > 3:
        x[2] = 0.25
        x[3, : L // 2] += 1e3                   # the first half salient: pieces of either list alone
    for k in (0, 1, L // 10, L // 2, L - 1, L):
        mask = torch.full((B, L), 7, dtype=torch.uint8, device="cuda")
        sal, reg = zb.zc_select_salient(x, k, mask=mask)
        first = torch.sort(x, dim=1, descending=True, stable=True).indices        # equal scores: lower index first
        assert torch.equal(sal.long(), first[:, :k].sort(dim=1).values) and torch.equal(reg.long(), first[:, k:].sort(dim=1).values)
        want = torch.zeros_like(mask).scatter_(1, first[:, :k], torch.ones_like(mask[:, :k]))
        assert torch.equal(mask, want)
