"""The head-wise budget allocation where heads are counted in several parts, where layers have more heads than are looked at
together, and where a head's safeguard ends among the keys that share the threshold's bin; and the one call's selection with
thresholds that the allocation leaves, by every route.  Budgets and indices against the oracle on the very scores
the library holds, so that both have to agree exactly."""
import numpy as np
import pytest

from oracle import curdkv_oracle as orc
from paper_2509_15038_amd import binding as B
from tests import gpu_util as gu

pytestmark = pytest.mark.gpu

PART = gu.limit("adaptive_kernels.hip", "kAdaPartTokens")
LIST = gu.limit("adaptive_kernels.hip", "kAdaList")
SEG = gu.limit("adaptive_kernels.hip", "kAdaSeg")                        # keys a head can have in the threshold's bin before the layer's scores are read again


def _heads(H, n, rng):
    """Heads of every temper: decades wide, flat, tied, one value, mostly zero, close to one another."""
    x = np.exp(rng.standard_normal((H, n)) * 2.0)
    for h in range(H):
        kind = h % 6
        if kind == 1:
            x[h] = 1.0 + rng.random(n) * 1e-2
        elif kind == 2:
            x[h] = np.round(rng.random(n) * 30) + 1
        elif kind == 3 and h > 6:
            x[h] = 1.0
        elif kind == 4:
            x[h, n // 3:] = 0.0
        elif kind == 5:
            x[h] = x[0]
    return (x / x.sum(1, keepdims=True)).astype(np.float32)


@pytest.mark.parametrize("L,H,n", [(1, 1, PART + 1), (2, 8, PART), (1, 8, PART + 1), (3, 3, 5 * PART - 7), (1, 9, 2 * PART + 1), (1, 17, 4500),
                                   (1, 2, 131072), (1, 64, 3000), (1, 65, 3000), (1, 300, 700), (2, 1024, 33), (40, 8, 300)])
def test_budgets(L, H, n):
    import torch
    rng = np.random.Generator(np.random.PCG64([L, H, n]))
    sc = np.stack([_heads(H, n, rng) for _ in range(L)])
    sc[L - 1] = sc[L - 1][rng.permutation(H)]
    dev = torch.from_numpy(sc.reshape(L * H, n)).cuda()
    out = torch.empty((L * H,), dtype=torch.int32, device="cuda")
    with B.Context(L, H, 4, 128, 32, "bf16", n, 1) as ctx:
        for k, s, alpha in ((n // 10, 4, 0.2), (n // 3, 0, 0.0), (n // 2, 4, 0.9), (n // 7, 64, 0.5), (n - 1, 4, 0.2), (5, 4, 0.2), (n // 4 + 1, 1, 1.0)):
            if not 0 <= k <= n:
                continue
            out.fill_(-7)
            ctx.adaptive_budgets(dev, n, k, s, alpha, out)
            got = out.cpu().numpy().reshape(L, H)
            for layer in range(L):
                assert got[layer].tolist() == orc.adaptive_budgets(sc[layer].astype(np.float64), k, s, alpha).tolist(), (layer, k, s, alpha)
            if L * H <= 1024:
                ctx.adaptive_budgets_noalloc(dev, n, k, s, alpha, out)
                assert out.cpu().numpy().tolist() == got.reshape(-1).tolist()


# keys in the threshold's bin: as many as the list and a head's segment take, and more; the safeguard ends above the bin, inside it, below it
@pytest.mark.parametrize("inside", [1, 31, 33, LIST // 4 - 1, LIST // 4, LIST // 4 + 1, 1920, 1921, SEG, SEG + 1])
def test_safeguard_inside_the_bin(inside):
    import torch
    H, n, above = 4, 20000, 100
    rng = np.random.Generator(np.random.PCG64([inside]))
    sc = rng.uniform(0.0, 0.2, (H, n)).astype(np.float32)
    for h in range(H):
        place = rng.permutation(n)
        sc[h, place[:above * (h + 1)]] = rng.uniform(1.1, 1.9, above * (h + 1))
        sc[h, place[above * (h + 1):above * (h + 1) + inside]] = 0.5 + rng.integers(0, 2 ** 18, inside) * 2.0 ** -24 * (1.0 if h != 2 else 0.0)
    dev = torch.from_numpy(sc).cuda()
    out = torch.empty((H,), dtype=torch.int32, device="cuda")
    with B.Context(1, H, 4, 128, 32, "bf16", n, 1) as ctx:
        for g in (50, above, above + inside // 2, above + inside, 3 * above + inside // 3, 2 * above + inside):
            for extra in (1, inside, 2 * inside):
                k = max(g + 1, (above * (1 + 2 + 3 + 4) + extra) // H)
                alpha = g / k
                ctx.adaptive_budgets(dev, n, k, 0, alpha, out)
                assert out.cpu().numpy().tolist() == orc.adaptive_budgets(sc.astype(np.float64), k, 0, alpha).tolist(), (g, extra)


# (selection and gather in one launch; by one workgroup per head; by several; streamed; 256 heads: scored by the fused kernel)
@pytest.mark.parametrize("L,H,n,dtype", [(1, 1, 257, "bf16"), (1, 8, 300, "fp32"), (1, 8, 4097, "bf16"), (2, 5, 32768, "bf16"), (1, 8, 32769, "bf16"),
                                         (1, 8, 36865, "bf16"), (1, 2, 131072, "bf16"), (1, 3, 70000, "fp32"), (5, 8, 40001, "bf16"), (33, 4, 37000, "bf16"),
                                         (32, 8, 600, "bf16")])
@pytest.mark.parametrize("alpha", [0.2, 0.9])
def test_one_call(L, H, n, dtype, alpha):
    import torch
    heads, s = L * H, 4
    g = torch.Generator(device="cuda")
    g.manual_seed(n)
    dt = torch.bfloat16 if dtype == "bf16" else torch.float32
    K = torch.empty((heads, n, 128), dtype=dt, device="cuda")
    V = torch.empty_like(K)
    for h in range(heads):                                              # every other head flat: it keeps its safeguard alone
        K[h] = torch.randn((n, 128), generator=g, device="cuda")
        V[h] = torch.randn((n, 128), generator=g, device="cuda") * (torch.randn((n, 1), generator=g, device="cuda") * 3).exp() if h % 2 == 0 else 1.0
    k = n // 10 + 5
    with B.Context(L, H, 4, 128, 20, dtype, n, 7) as ctx:
        sc = gu.Guarded((heads, n), torch.float32, float("nan"))
        bud = gu.Guarded((heads,), torch.int32, -7)
        off = gu.Guarded((heads + 1,), torch.int64, -7)
        idx = gu.Guarded((heads * k,), torch.int32, -7)
        Ko, Vo = gu.Guarded((heads * k, 128), dt, float("nan")), gu.Guarded((heads * k, 128), dt, float("nan"))
        for _ in range(2):                                              # the second on what the first left in the workspace
            ctx.compress_adaptive(K, V, n, k, s, alpha, sc.t, bud.t, off.t, idx.t, Ko.t, Vo.t)
        torch.cuda.synchronize()
        for x in (sc, bud, off, idx, Ko, Vo):
            x.check()
        apart = torch.empty((heads, n), dtype=torch.float32, device="cuda")
        ctx.scores(K, V, n, apart)
        assert torch.allclose(sc.t, apart, rtol=1e-6, atol=0)
    scores, budgets, offsets = sc.t.cpu().numpy().astype(np.float64), bud.t.cpu().numpy(), off.t.cpu().numpy()
    assert offsets.tolist() == np.concatenate([[0], np.cumsum(budgets, dtype=np.int64)]).tolist()
    where = idx.t.long()
    got = where.cpu().numpy()
    for layer in range(L):
        rows = slice(layer * H, (layer + 1) * H)
        assert budgets[rows].tolist() == orc.adaptive_budgets(scores[rows], k, s, alpha).tolist(), layer
        for h in range(layer * H, (layer + 1) * H):
            a, b = int(offsets[h]), int(offsets[h + 1])
            assert np.array_equal(got[a:b], orc.select(scores[h], int(budgets[h]), s)), h
            assert torch.equal(Ko.t[a:b], K[h, where[a:b]]) and torch.equal(Vo.t[a:b], V[h, where[a:b]]), h


def test_more_heads_than_a_grid_is_high():
    """66000 (layer, head) pairs, each its own workgroup."""
    import torch
    L, H, n = 16500, 4, 20
    rng = np.random.default_rng(5)
    sc = rng.random((L, H, n)).astype(np.float32)
    out = torch.full((L * H,), -7, dtype=torch.int32, device="cuda")
    with B.Context(L, H, 4, 128, 1, "bf16", n, 1) as ctx:
        ctx.adaptive_budgets(torch.from_numpy(sc.reshape(L * H, n)).cuda(), n, 7, 2, 0.5, out)
        got = out.cpu().numpy().reshape(L, H)
    for layer in (0, 1, 8000, 16383, 16384, L - 1):
        assert got[layer].tolist() == orc.adaptive_budgets(sc[layer].astype(np.float64), 7, 2, 0.5).tolist(), layer
    assert np.all(got.sum(1) == 7 * H)
