"""Few, short heads in one call: the selection whose workgroups copy their share of the rows.  Indices against the oracle's
selection on the very scores the library stored, rows against torch's indexing, scores against the separate calls."""
import numpy as np
import pytest

from oracle import curdkv_oracle as orc
from paper_2509_15038_amd import binding as B
from paper_2509_15038_amd import workloads as wl
from tests import gpu_util as gu

pytestmark = pytest.mark.gpu

ROWS = gu.limit("select_kernels.hip", "kGatherRowsPerUnit") * 256       # rows kept, all heads, up to which this route is taken
LONGEST = 32 * gu.limit("select_kernels.hip", "kSelThreads")            # the longest head that a workgroup's registers hold


def _cache(heads, n, dtype, seed):
    import torch
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    K, V = (torch.randn((heads, n, 128), generator=g, device="cuda") * torch.randn((heads, n, 1), generator=g, device="cuda").exp() for _ in range(2))
    if heads > 1:
        V[1] = V[1, :1]                                       # rows of one value: every candidate ties,
        K[1] = K[1, :1]
    if heads > 2:
        V[2] = 0                                              # scores of 1/n,
    if heads > 4:
        K[4, n // 3:] = K[4, n // 3].clone()                  # and a stretch of equal scores
        V[4, n // 3:] = V[4, n // 3].clone()
    dt = torch.bfloat16 if dtype == "bf16" else torch.float32
    return (x.to(dt).view(1, heads, n, 128) for x in (K, V))


def _check(heads, n, dtype, budgets, s, r=20, source="kv", projection=True, seed=3):
    import torch
    budgets = np.minimum(np.asarray(budgets), n).astype(np.int32)
    K, V = _cache(heads, n, dtype, seed)
    with B.Context(1, heads, 4, 128, r, dtype, n, 77, source, projection) as ctx:
        sc, idx, Ko, Vo, off = gu.run_path(ctx, K, V, n, budgets, s, dtype, one_call=True)
        apart = torch.empty_like(sc)
        ctx.scores(K, V, n, apart)
        assert torch.allclose(sc, apart, rtol=1e-6, atol=0)            # (the sum is added in the same order or not: 2^-24 each)
        scores, where = sc.cpu().numpy().astype(np.float64), idx.long()
        got = where.cpu().numpy()
        for h in range(heads):
            a, b = int(off[h]), int(off[h + 1])
            assert np.array_equal(got[a:b], orc.select(scores[h], int(budgets[h]), s)), (h, int(budgets[h]))
            assert torch.equal(Ko[a:b], K[0, h, where[a:b]]) and torch.equal(Vo[a:b], V[0, h, where[a:b]]), h
        # without the scores the rows are the same ones
        i2, k2, v2 = (torch.zeros_like(x) for x in (idx, Ko, Vo))
        ctx.compress(K, V, n, budgets, s, off, None, i2, k2, v2)
        assert torch.equal(i2, idx) and torch.equal(k2, Ko) and torch.equal(v2, Vo)


# (lengths at the edges of the bitmap's words, of a thread's 4, 8, 16 and 32 keys, and of the route)
@pytest.mark.parametrize("dtype", ["bf16", "fp32"])
@pytest.mark.parametrize("heads,n", [(1, 1), (1, 63), (5, 65), (6, 1000), (3, 1024), (8, 4096), (8, 4097), (5, 8193), (7, 16385), (3, LONGEST), (128, 300), (100, 1023)])
def test_budgets_of_every_kind(heads, n, dtype):
    kinds = [n // 5, n // 3 + 1, 1, 0, n, n - 1, 5, 64, 65]   # some heads keep next to nothing, some everything
    for s in (0, 4, 64):
        _check(heads, n, dtype, [kinds[h % len(kinds)] for h in range(heads)], s)
    _check(heads, n, dtype, [n // 4 + 1] * heads, 4, r=64, seed=9)


@pytest.mark.parametrize("source,projection", [("k", True), ("v", True), ("kv", False)])
def test_other_scores(source, projection):
    _check(6, 1500, "bf16", [300] * 6, 4, source=source, projection=projection)


# budgets on both sides of the limit of rows, heads on both sides of the limit of tokens (33: more than the split selection takes
# below 36864 tokens)
@pytest.mark.parametrize("heads,n,total", [(33, LONGEST, 33 * 200), (33, LONGEST + 1, 33 * 200), (32, LONGEST, 32 * 200), (3, LONGEST + 1, 3 * 2000), (64, 8192, ROWS),
                                           (64, 8192, ROWS + 64), (128, 2048, ROWS)])
def test_both_sides_of_the_rule(heads, n, total):
    _check(heads, n, "bf16", [total // heads] * heads, 4)


def test_nothing_kept():
    """All budgets zero: scores only."""
    _check(4, 2000, "bf16", [0] * 4, 4)


@pytest.mark.parametrize("n", [1, 2, 65, 1025, 24577, 32768])
def test_heads_without_a_sum(n):
    """A head of zeros, and one whose sum is not a number: every score is 1/n, and the first tokens are kept."""
    import torch
    heads = 6
    K, V = _cache(heads, n, "bf16", 5)
    V[0, 1], K[0, 3] = 0, 0
    V[0, 4, n // 2] = float("nan")
    budgets = np.minimum([n // 3 + 1, n // 10 + 5, n // 7, n - 1, n // 5 + 2, 3], n).astype(np.int32)
    with B.Context(1, heads, 4, 128, 20, "bf16", n, 77) as ctx:
        for b in (budgets, np.full((heads,), n, np.int32), np.full((heads,), min(4, n), np.int32)):
            sc, idx, Ko, Vo, off = gu.run_path(ctx, K, V, n, b, 4, "bf16", one_call=True)
            where = idx.long()
            for h in range(heads):
                a, z = int(off[h]), int(off[h + 1])
                if h in (1, 3, 4):
                    assert bool((sc[h] == np.float32(1.0 / n)).all()) and where[a:z].tolist() == list(range(z - a)), h
                assert np.array_equal(where[a:z].cpu().numpy(), orc.select(sc[h].cpu().numpy().astype(np.float64), int(b[h]), 4)), h
                bits = torch.int16
                assert torch.equal(Ko[a:z].view(bits), K[0, h, where[a:z]].view(bits)) and torch.equal(Vo[a:z].view(bits), V[0, h, where[a:z]].view(bits)), h


# the longest head of every number of keys per thread, and one token more
@pytest.mark.parametrize("keys", [1, 2, 3, 4, 6, 8, 10, 12, 14, 16, 20, 24, 28, 32])
@pytest.mark.parametrize("more", [0, 1])
def test_keys_per_thread(keys, more):
    import torch
    n = 1024 * keys + more
    rng = np.random.default_rng(n)
    scores = np.exp(rng.standard_normal((3, n)) * 2).astype(np.float32)
    scores[1] = np.round(rng.random(n) * 50)
    scores[2, :-1] = 0.0
    budgets = np.array([n // 10, n // 3, n - 5], dtype=np.int32)
    off = wl.offsets_for(budgets)
    with B.Context(1, 3, 4, 128, 20, "bf16", n, 1) as ctx:
        out = gu.Guarded((int(off[-1]),), torch.int32, -7)
        ctx.select(torch.from_numpy(scores).cuda(), n, budgets, 4, off, out.t)
        got = out.t.cpu().numpy()
        out.check()
    for h in range(3):
        assert np.array_equal(got[off[h]:off[h + 1]], orc.select(scores[h].astype(np.float64), int(budgets[h]), 4)), h
    if keys in (1, 3, 10, 24, 32):
        _check(2, n, "bf16", [n // 10, n // 7], 4)


# (33000: one workgroup's indices, 4 bytes a token, need more LDS than a launch gets by itself, as 14000's and 20000's do; 9000's do not)
@pytest.mark.parametrize("heads,n", [(3, 9000), (3, 14000), (3, 20000), (40, 33000)])
def test_captured(heads, n):
    """One call and the selection in a graph, replayed on other caches, against the same calls without one."""
    import torch
    budgets = np.full((heads,), n // 10, np.int32)
    off = wl.offsets_for(budgets)
    total = int(off[-1])
    K, V = (x.clone() for x in _cache(heads, n, "bf16", 1))
    with B.Context(1, heads, 4, 128, 20, "bf16", n, 77) as ctx:
        def buffers():
            return [torch.empty((heads, n), device="cuda"), torch.empty((total,), dtype=torch.int32, device="cuda"),
                    torch.empty((total, 128), dtype=K.dtype, device="cuda"), torch.empty((total, 128), dtype=K.dtype, device="cuda"),
                    torch.empty((total,), dtype=torch.int32, device="cuda")]

        def calls(sc, ix, Ko, Vo, again):
            ctx.compress(K, V, n, budgets, 4, off, sc, ix, Ko, Vo)
            ctx.select(sc, n, budgets, 4, off, again)

        kept, eager = buffers(), buffers()
        calls(*kept)
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph):
            calls(*kept)
        for seed in (2, 3, 4):
            for mine, new in zip((K, V), _cache(heads, n, "bf16", seed)):
                mine.copy_(new)
            for x in kept:
                x.fill_(-1)
            graph.replay()
            torch.cuda.synchronize()
            calls(*eager)
            torch.cuda.synchronize()
            for a, b in zip(kept, eager):
                assert torch.equal(a, b), seed
            assert torch.equal(kept[1], kept[4]), seed


# the heads along x, so that a head's workgroups meet in one L2, from 2049 tokens on, and up to 8192 only where fewer than a quarter of the rows are kept
@pytest.mark.parametrize("heads,n,budget,heads_x", [(12, 2048, 400, False), (12, 2049, 400, True), (12, 4096, 1023, True), (12, 4096, 1024, False), (5, 8192, 4000, False), (5, 8193, 4000, True)])
def test_order_of_the_grid(heads, n, budget, heads_x):
    import torch
    budgets = np.full((heads,), budget, np.int32)
    K, V = _cache(heads, n, "bf16", 4)
    with B.Context(1, heads, 4, 128, 20, "bf16", n, 77) as ctx:
        sc, idx, Ko, Vo, off = gu.run_path(ctx, K, V, n, budgets, 4, "bf16", one_call=True)
        name, _, grid = gu.launches(lambda: ctx.compress(K, V, n, budgets, 4, off, sc, idx, Ko, Vo))[-1]
    assert name == "select_gather_kernel" and grid[1 - heads_x] == heads and grid[int(heads_x)] != heads, grid
    where = idx.long()
    for h in range(heads):
        mine = slice(int(off[h]), int(off[h + 1]))
        assert np.array_equal(where[mine].cpu().numpy(), orc.select(sc[h].cpu().numpy().astype(np.float64), budget, 4)), h
        assert torch.equal(Ko[mine], K[0, h, where[mine]]) and torch.equal(Vo[mine], V[0, h, where[mine]]), h
