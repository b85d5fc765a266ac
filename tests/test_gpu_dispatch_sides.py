"""Kernels that are reached only beyond a dispatch limit, at sizes taken from that limit: fp32 scoring of more
tokens than the kernel for few takes, the streaming selection in more heads than the split one takes, and the
split selection's one-call variants.  Against the float64 oracle."""
import numpy as np
import pytest

from oracle import curdkv_oracle as orc
from paper_2509_15038_amd import binding as B
from paper_2509_15038_amd import workloads as wl
from tests import gpu_util as gu

pytestmark = pytest.mark.gpu

SEED = 0xC0DE0013
FEW_F32 = gu.limit("scores_kernels.hip", "kFewF32Tokens")
FEW_HEADS_F32 = gu.limit("scores_kernels.hip", "kFewHeadsF32")
SPLIT_HEADS = gu.limit("curdkv_internal.h", "kSplitMaxHeads")
SPLIT_FROM_ELSE = gu.limit("split_select.hip", "kSplitMinTokensElse")
GATHER_LONGEST = 32 * gu.limit("select_kernels.hip", "kSelThreads")     # up to here few heads take the selection that gathers

# A projected coordinate takes 32 roundings of a sum of 128 products (one per 4 products in fp32; one per 32 over six
# passes of split products, and 2^-24 per product at most left out), at random; squared and summed over r,
# multiplied and normalised: some 30 roundings of 2^-24 relative to the score
NORM_TOL = 1e-6


# edges of the 16-token steps, the 32-token tiles, the 64-token groups and of a wave's range; plain fp32 products (r <= 32)
# and split ones
@pytest.mark.parametrize("n", [15, 17, 31, 33, 63, 64, 65, 127, 300, 1009])
@pytest.mark.parametrize("r,source", [(20, "kv"), (20, "k"), (32, "v"), (33, "kv"), (64, "k"), (65, "v"), (128, "kv")])
def test_f32_scores_beyond_the_few(n, r, source):
    import torch
    heads = FEW_F32 // n + 1
    if r <= 32:                                          # (the kernel for few tokens takes more of these, by its load, in up to so many heads)
        heads = max(heads, FEW_HEADS_F32 + 1) if n < 1000 else 64
    g = torch.Generator(device="cuda")
    g.manual_seed(n * 512 + r)
    K = torch.randn((heads, n, 128), generator=g, device="cuda") * torch.exp(torch.randn((heads, 1, 128), generator=g, device="cuda"))
    V = torch.randn((heads, n, 128), generator=g, device="cuda") * torch.exp(torch.randn((heads, n, 1), generator=g, device="cuda"))
    with B.Context(heads, 1, 4, 128, r, "fp32", n, SEED, source) as ctx:
        out = torch.full((heads, n), float("nan"), device="cuda")
        ctx.scores(K, V, n, out)
        name, args, _ = gu.launches(lambda: ctx.scores(K, V, n, out))[0]
        assert name == "scores_f32_kernel" and args[4] == (r > 32), (name, args)
        torch.cuda.synchronize()
        raw, sums = torch.full((heads, n), float("nan"), device="cuda"), torch.zeros((heads,), dtype=torch.float64, device="cuda")
        ctx.scores_append(K, V, n, 0, n, raw, sums)
        out, raw, sums = out.cpu().numpy(), raw.cpu().numpy().astype(np.float64), sums.cpu().numpy()
    assert np.allclose(sums, raw.sum(1), rtol=1e-6)
    for i in (0, heads // 2, heads - 1):
        G = orc.sketch(SEED, i, 0, 1, 128, r, "fp32")
        want = orc.scores(K[i].double().cpu().numpy(), V[i].double().cpu().numpy(), G, source)
        for x in (out[i], raw[i] / raw[i].sum()):
            assert np.linalg.norm(x - want) <= NORM_TOL * np.linalg.norm(want), (n, r, source, i)


# (widths without columns of padding, whose zeros make an infinity a NaN in any order; up to 32 columns the split products begin at a number of tokens)
@pytest.mark.parametrize("r,heads", [(32, 1024), (64, FEW_F32 // 300 + 1), (128, FEW_F32 // 300 + 1)])
@pytest.mark.parametrize("source", ["kv", "k", "v"])
def test_f32_rows_that_are_not_finite_beyond_the_few(r, heads, source):
    import torch
    n = 300
    g = torch.Generator(device="cuda")
    g.manual_seed(r)
    K, V = torch.randn((heads, n, 128), generator=g, device="cuda"), torch.randn((heads, n, 128), generator=g, device="cuda")

    def raw_scores():
        with B.Context(heads, 1, 4, 128, r, "fp32", n, SEED, source) as ctx:
            raw, sums = torch.full((heads, n), -1.0, device="cuda"), torch.zeros((heads,), dtype=torch.float64, device="cuda")
            call = lambda: ctx.scores_append(K, V, n, 0, n, raw, sums)
            call()
            name, args, _ = gu.launches(call)[0]
            assert name == "scores_f32_kernel" and args[4] == 1, (name, args)
            return raw.cpu().numpy()

    clean = raw_scores()
    K[1, 5, 17] = float("inf")
    K[1, 130, 3] = float(np.finfo(np.float32).max)
    V[1, 77, 100] = float("nan")
    V[1, 299, 0] = -float("inf")
    raw = raw_scores()
    infinite, nan = [j for j, of in ((5, "k"), (130, "k"), (299, "v")) if of in source], [77] if "v" in source else []
    assert np.all(np.isposinf(raw[1, infinite])) and np.all(np.isnan(raw[1, nan]))
    clean[1, infinite + nan] = raw[1, infinite + nan] = 0.0
    assert np.array_equal(raw, clean)


# rows that the bf16 parts do not hold, scored again after the walk, where the scan also counts for the split selection
@pytest.mark.parametrize("r", [32, 64])
def test_one_call_with_rows_at_the_top_of_the_range(r):
    """A channel of the largest floats under a sketch of 2^-80: the rows' first parts are infinite, their scores are not, and are the largest."""
    import torch
    heads, n, s = 4, 70001, 4
    g = torch.Generator(device="cuda")
    g.manual_seed(r)
    K = torch.randn((heads, n, 128), generator=g, device="cuda")
    V = torch.randn((heads, n, 128), generator=g, device="cuda") * torch.randn((heads, n, 1), generator=g, device="cuda").exp()
    K[..., 17] = 0
    top = torch.tensor([3, 4, 63, 64, 30000, 30031, 44444, n - 1], device="cuda")
    K[1, top, 17] = float(np.finfo(np.float32).max)
    K[3, top, 17] = -float(np.finfo(np.float32).max)
    G = np.stack([orc.sketch(SEED, 0, h, heads, 128, r, "fp32") for h in range(heads)])
    G[:, 17] = np.sign(G[:, 17]) * 2.0 ** -80
    budgets = np.array([n // 10, n // 10, n // 3, 9], np.int32)
    with B.Context(1, heads, 4, 128, r, "fp32", n, SEED) as ctx:
        for h in range(heads):
            ctx.set_sketch(0, h, G[h].astype(np.float32))
        sc, ix, Ko, Vo, off = gu.run_path(ctx, K, V, n, budgets, s, "fp32", one_call=True)
        name, args, _ = gu.launches(lambda: ctx.compress(K, V, n, budgets, s, off, sc, ix, Ko, Vo))[0]
        torch.cuda.synchronize()
    assert name == "scores_f32_kernel" and args[3:5] == (1, 1), (name, args)
    for h in range(heads):
        lt = orc.scores(K[h].double().cpu().numpy(), V[h].double().cpu().numpy(), G[h])
        rows = ix[off[h]:off[h + 1]].cpu().numpy().astype(np.int64)
        gu.check_scores(sc[h].cpu().numpy(), lt, str(h))
        gu.check_selection(rows, lt, int(budgets[h]), s, str(h))
        if h in (1, 3):
            assert np.isin(top.cpu().numpy(), rows).sum() >= (8 if h == 1 else 5)          # (of head 3 five beside the sinks, of which 3 is one)
        assert torch.equal(Ko[off[h]:off[h + 1]], K[h, rows]) and torch.equal(Vo[off[h]:off[h + 1]], V[h, rows])


def _full_bin(rng, n, in_bin):
    """Scores of which `in_bin` share the bin [1, 1 + 1/32), n / 50 lie above it and the rest far below."""
    sc = rng.random(n).astype(np.float32) * np.float32(0.4) + np.float32(1e-3)
    where = rng.permutation(n)
    sc[where[:in_bin]] = np.float32(1.0) + rng.integers(0, max(in_bin // 3, 2), size=in_bin).astype(np.float32) * np.float32(2.0 ** -23)
    sc[where[in_bin:in_bin + n // 50]] = np.float32(1.5) + rng.random(n // 50).astype(np.float32) * np.float32(0.4)
    return sc, n // 50


# one workgroup per head streams the scores: a list of 8192 keys, and one more; a bitmap block of 131072 tokens, and more
@pytest.mark.parametrize("n,in_bin", [(SPLIT_FROM_ELSE + 1, 100), (60000, 8191), (60000, 8192), (60000, 8193), (131072, 8192), (131073, 8193)])
def test_streaming_selection_in_many_heads(n, in_bin):
    import torch
    rng = np.random.default_rng([n, in_bin])
    heads, s = SPLIT_HEADS + 1, 4
    sc = np.tile(rng.random(n).astype(np.float32), (heads, 1))
    budgets = np.full((heads,), 5, np.int32)
    for i, h in enumerate((0, 1, 77, heads - 1)):
        sc[h], above = _full_bin(rng, n, in_bin)
        budgets[h] = s + above + [1, in_bin // 2, in_bin, 1 + in_bin // 3][i]      # cut at the top, inside and at the bottom of the bin
    sc[5] = (rng.integers(0, 50, n) * 1e-6).astype(np.float32)                     # ties everywhere
    budgets[5] = n // 3
    off = wl.offsets_for(budgets)
    with B.Context(1, heads, 4, 128, 64, "bf16", n, 1) as ctx:
        idx = gu.Guarded((int(off[-1]),), torch.int32, -1)
        ctx.select(torch.from_numpy(sc).cuda(), n, budgets, s, off, idx.t)
        torch.cuda.synchronize()
        idx.check("indices")
        idx = idx.t.cpu().numpy()
    for h in (0, 1, 5, 77, 100, heads - 1):
        assert np.array_equal(idx[off[h]:off[h + 1]], orc.select(sc[h].astype(np.float64), int(budgets[h]), s)), (n, in_bin, h)


# every scoring kernel that counts for the split selection: storage, width, source, no projection; scores, indices and rows
@pytest.mark.parametrize("dtype,r,source,projection", [("bf16", 20, "kv", True), ("bf16", 64, "k", True), ("bf16", 128, "v", True), ("bf16", 64, "kv", False),
                                                       ("bf16", 64, "k", False), ("fp32", 20, "kv", True), ("fp32", 32, "v", True), ("fp32", 64, "k", True),
                                                       ("fp32", 128, "kv", True), ("fp32", 64, "kv", False), ("fp32", 64, "v", False)])
def test_one_call_of_long_heads(dtype, r, source, projection):
    n = GATHER_LONGEST + 1213
    cfg = wl.scaled(wl.CONFIGS["c2"], kv_heads=3, n=n, r=r, dtype=dtype)
    budgets = np.array([n // 10, n // 2, 67], dtype=np.int32)
    gu.run_and_check(cfg, budgets, one_call=True, source=source, projection=projection, fused=False)


@pytest.mark.parametrize("heads,n,r", [(33, SPLIT_FROM_ELSE + 1, 20), (2, 131072, 64)])
def test_one_call_of_long_heads_at_the_ends(heads, n, r):
    cfg = wl.scaled(wl.CONFIGS["c2"], kv_heads=heads, n=n, r=r)
    budgets = np.full((heads,), n // 9, dtype=np.int32)
    gu.run_and_check(cfg, budgets, one_call=True, fused=False)


@pytest.mark.parametrize("dtype", ["bf16", "fp32"])
def test_one_call_with_more_rows_than_the_split_gathers(dtype):
    """From 1024 kept rows per compute unit on, the gather is a kernel of its own."""
    import torch
    rows = 1024 * torch.cuda.get_device_properties(0).multi_processor_count
    heads, n, s = 8, 40000, 4
    cfg = wl.scaled(wl.CONFIGS["c2"], kv_heads=heads, n=n, r=20, dtype=dtype)
    K, V = wl.host_cache(cfg)
    for total in (rows, rows + 1):
        budgets = np.full((heads,), total // heads, dtype=np.int32)
        budgets[0] += total - int(budgets.sum())
        if budgets.max() > n:
            pytest.skip("more compute units than this test has rows for")
        gu.run_and_check(cfg, budgets, K=K, V=V, one_call=True, fused=False)
        off = wl.offsets_for(budgets)
        Kd, Vd = gu.to_device(K, dtype), gu.to_device(V, dtype)
        with B.Context(1, heads, 4, 128, 20, dtype, n, cfg.sketch_seed) as ctx:
            sc = torch.empty((heads, n), device="cuda")
            ix, ix2 = torch.empty((total,), dtype=torch.int32, device="cuda"), torch.full((total,), -7, dtype=torch.int32, device="cuda")
            Ko, Vo = torch.empty((total, 128), dtype=Kd.dtype, device="cuda"), torch.empty((total, 128), dtype=Kd.dtype, device="cuda")
            Ko2, Vo2 = torch.full_like(Ko, float("nan")), torch.full_like(Vo, float("nan"))
            ctx.compress(Kd, Vd, n, budgets, s, off, sc, ix, Ko, Vo)
            ctx.compress(Kd, Vd, n, budgets, s, off, None, ix2, Ko2, Vo2)
            assert torch.equal(ix, ix2) and torch.equal(Ko, Ko2) and torch.equal(Vo, Vo2)


LONG_FROM = gu.limit("curdkv_internal.h", "kFusedGatherTokens")
SHARE = gu.limit("curdkv_internal.h", "kFusedGatherLongShare")
CACHED_FROM = gu.limit("scores_kernels.hip", "kStartHeadBytes") // 512 + 1
UNEVEN, UNEVEN_LONG, UNEVEN_ROUNDS = (gu.limit("curdkv_internal.h", "kFusedUnevenRows" + which) for which in ("", "Long", "Rounds"))


# budgets whose largest is a row beyond what one workgroup copies alone, and not, the average within the fused kernel's limit; equal ones on both sides of that limit, where the scan's start
# goes through the caches and where it does not
@pytest.mark.parametrize("rounds,n,average,more,fused", [(1, LONG_FROM, 300, UNEVEN, True), (1, LONG_FROM, 300, UNEVEN + 1, False), (1, 1111, 500, UNEVEN + 1, False), (1, 700, 300, 400, True),
                                                         (1, LONG_FROM + 1, 300, UNEVEN_LONG, True), (1, LONG_FROM + 1, 300, UNEVEN_LONG + 1, False),
                                                         (2, 801, 390, UNEVEN_ROUNDS, True), (2, 801, 390, UNEVEN_ROUNDS + 1, False),
                                                         (1, CACHED_FROM, CACHED_FROM // SHARE, 0, True), (1, CACHED_FROM, CACHED_FROM // SHARE + 1, 0, False), (1, CACHED_FROM - 1, CACHED_FROM // SHARE + 1, 0, True)])
def test_fused_gather_of_uneven_budgets(rounds, n, average, more, fused):
    import torch
    heads, s = rounds * torch.cuda.get_device_properties(0).multi_processor_count, 4
    g = torch.Generator(device="cuda")
    g.manual_seed(n)
    K = torch.randn((heads, n, 128), generator=g, device="cuda").to(torch.bfloat16)
    V = (torch.randn((heads, n, 128), generator=g, device="cuda") * torch.randn((heads, n, 1), generator=g, device="cuda").exp()).to(torch.bfloat16)
    budgets = np.full((heads,), average, np.int32)
    budgets[5] += more
    budgets[7] -= min(more, average)
    budgets[9] -= more - min(more, average)                                # the average stays
    with B.Context(1, heads, 4, 128, 64, "bf16", n, SEED) as ctx:
        sc, ix, Ko, Vo, off = gu.run_path(ctx, K, V, n, budgets, s, "bf16", one_call=True)
        names = [name for name, _, _ in gu.launches(lambda: ctx.compress(K, V, n, budgets, s, off, sc, ix, Ko, Vo))]
        torch.cuda.synchronize()
    assert (names == ["fused_kernel"]) == fused and names[0] == "fused_kernel", names
    sc, rows = sc.cpu().numpy().astype(np.float64), ix.long()
    for h in (0, 5, 7, 9, heads - 1):
        mine = slice(int(off[h]), int(off[h + 1]))
        assert np.array_equal(rows[mine].cpu().numpy(), orc.select(sc[h], int(budgets[h]), s)), h
        assert torch.equal(Ko[mine], K[h, rows[mine]]) and torch.equal(Vo[mine], V[h, rows[mine]]), h


def test_uneven_budgets_captured_before_any_scratch_for_scores():
    """The call with scores has uploaded the offsets; the same without scores is captured before it has ever run: by the one kernel, which allocates nothing."""
    import torch
    heads, n, s = torch.cuda.get_device_properties(0).multi_processor_count, 1024, 4
    g = torch.Generator(device="cuda")
    g.manual_seed(n)
    K = torch.randn((heads, n, 128), generator=g, device="cuda").to(torch.bfloat16)
    V = (torch.randn((heads, n, 128), generator=g, device="cuda") * torch.randn((heads, n, 1), generator=g, device="cuda").exp()).to(torch.bfloat16)
    budgets = np.full((heads,), 200, np.int32)
    budgets[3] += UNEVEN + 1
    off = np.concatenate([[0], np.cumsum(budgets, dtype=np.int64)])
    with B.Context(1, heads, 4, 128, 64, "bf16", n, SEED) as ctx:
        sc = torch.empty((heads, n), dtype=torch.float32, device="cuda")
        ix = torch.empty((int(off[-1]),), dtype=torch.int32, device="cuda")
        Ko, Vo = torch.empty((int(off[-1]), 128), dtype=K.dtype, device="cuda"), torch.empty((int(off[-1]), 128), dtype=K.dtype, device="cuda")
        ix2, Ko2, Vo2 = torch.empty_like(ix), torch.empty_like(Ko), torch.empty_like(Vo)
        ctx.compress(K, V, n, budgets, s, off, sc, ix, Ko, Vo)
        torch.cuda.synchronize()
        assert [name for name, _, _ in gu.launches(lambda: ctx.compress(K, V, n, budgets, s, off, None, ix2, Ko2, Vo2))] == ["fused_kernel"]
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph):
            ctx.compress(K, V, n, budgets, s, off, None, ix2, Ko2, Vo2)
        for _ in range(3):
            for t in (ix2, Ko2, Vo2):
                t.zero_()
            graph.replay()
            torch.cuda.synchronize()
            assert torch.equal(ix, ix2) and torch.equal(Ko, Ko2) and torch.equal(Vo, Vo2)
        del graph
