"""Scoring of more rows than the caches hold, which are fetched by whole lines past them: at sizes taken from that limit,
at the edges of the 16-token steps, the 32-token tiles and a wave's range.  Against the float64 oracle."""
import numpy as np
import pytest

from oracle import curdkv_oracle as orc
from paper_2509_15038_amd import binding as B
from paper_2509_15038_amd import workloads as wl
from tests import gpu_util as gu

pytestmark = pytest.mark.gpu

SEED = 0xC0DE0014
LIMIT = gu.limit("scores_kernels.hip", "kStreamBytes")
LIMIT_REREAD = gu.limit("scores_kernels.hip", "kStreamBytesReread")
LIMIT_REREAD_MANY = gu.limit("scores_kernels.hip", "kStreamBytesRereadMany")

# A projected coordinate is an fp32 sum of 128 exact products, rounded once per 32 terms, its square and their sum over r columns as many
# roundings again, then a product and the division: some 30 roundings of 2^-24 at random, relative to the score
NORM_TOL = 1e-6


def _heads(limit, n, dtype, source):
    return limit // (n * 128 * (2 if dtype == "bf16" else 4) * (2 if source == "kv" else 1)) + 1


def _cache(heads, n, dtype, seed):
    import torch
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    dt = torch.bfloat16 if dtype == "bf16" else torch.float32
    K = torch.randn((heads, n, 128), generator=g, device="cuda") * torch.exp(torch.randn((heads, 1, 128), generator=g, device="cuda"))
    V = torch.randn((heads, n, 128), generator=g, device="cuda") * torch.exp(torch.randn((heads, n, 1), generator=g, device="cuda"))
    return K.to(dt), V.to(dt)


def _want(K, V, i, r, dtype, source, projection):
    G = orc.sketch(SEED, i, 0, 1, 128, r, dtype)
    return orc.scores(K[i].double().cpu().numpy(), V[i].double().cpu().numpy(), G, source, projection)


@pytest.mark.parametrize("n", [257, 300, 1009, 1024, 4133, 70001])
@pytest.mark.parametrize("dtype,r,source,projection", [("bf16", 20, "kv", True), ("bf16", 33, "k", True), ("bf16", 64, "v", True), ("bf16", 64, "kv", True),
                                                       ("bf16", 128, "kv", True), ("bf16", 64, "kv", False)])
def test_scores(n, dtype, r, source, projection):
    _check_scores(_heads(LIMIT, n, dtype, source), n, dtype, r, source, projection)


# up to 32 columns of an fp32 cache over the bf16 units: a group of 64 tokens a wave and more, whole groups and parts
@pytest.mark.parametrize("heads,n", [(2100, 63), (128, 1024), (1024, 300), (256, 1009), (100, 4133), (4, 70001)])
@pytest.mark.parametrize("r,source", [(20, "kv"), (32, "k"), (8, "v")])
def test_scores_of_narrow_sketches_in_fp32(heads, n, r, source):
    _check_scores(heads, n, "fp32", r, source, True)


def _check_scores(heads, n, dtype, r, source, projection):
    import torch
    K, V = _cache(heads, n, dtype, n * 512 + r)
    with B.Context(heads, 1, 4, 128, r, dtype, n, SEED, source, projection) as ctx:
        out = gu.Guarded((heads, n), torch.float32, float("nan"))
        ctx.scores(K, V, n, out.t)
        raw, sums = torch.full((heads, n), float("nan"), device="cuda"), torch.zeros((heads,), dtype=torch.float64, device="cuda")
        ctx.scores_append(K, V, n, 0, n, raw, sums)
        out.check("scores")
        out, raw, sums = out.t.cpu().numpy(), raw.cpu().numpy().astype(np.float64), sums.cpu().numpy()
    assert np.allclose(sums, raw.sum(1), rtol=1e-6)
    for i in (0, heads // 2, heads - 1):
        want = _want(K, V, i, r, dtype, source, projection)
        for x in (out[i], raw[i] / raw[i].sum()):
            assert np.linalg.norm(x - want) <= NORM_TOL * np.linalg.norm(want), (n, r, source, i)


# one call: the kernel that does everything (few rows kept of as many heads as units), scores by it and separate kernels, the selection
# that gathers, the split selection with histograms from the scoring; a quarter and more kept, where the end of the scan goes through the caches,
# is a walk in two parts.  The rows kept are found again
@pytest.mark.parametrize("heads,n,r,keep,dtype", [(256, 2048, 64, 0.9, "bf16"), (256, 2047, 20, 0.5, "bf16"), (256, 2049, 64, 0.1, "bf16"), (256, 2500, 20, 0.05, "bf16"), (256, 2111, 64, 0.5, "bf16"), (25, 16411, 64, 0.1, "bf16"),
                                                  (32, 16411, 20, 0.3, "bf16"), (200, 2600, 20, 0.4, "bf16"), (6, 70001, 20, 0.1, "bf16"), (8, 70001, 64, 0.5, "bf16"),
                                                  (40, 40001, 128, 0.05, "bf16"), (11, 49217, 128, 0.6, "bf16"), (100, 4133, 20, 0.1, "fp32"), (4, 70001, 32, 0.4, "fp32"),
                                                  (256, 1009, 20, 0.5, "fp32")])
def test_one_call(heads, n, r, keep, dtype):
    import torch
    if heads == 256:
        heads = torch.cuda.get_device_properties(0).multi_processor_count
    assert heads * n * 512 > (LIMIT_REREAD if keep < 0.25 else LIMIT_REREAD_MANY) or dtype == "fp32" or n <= 2048
    K, V = _cache(heads, n, dtype, n + r)
    budgets = np.full((heads,), int(keep * n), np.int32)
    with B.Context(heads, 1, 4, 128, r, dtype, n, SEED) as ctx:
        sc, ix, Ko, Vo, off = gu.run_path(ctx, K, V, n, budgets, 4, dtype, one_call=True)
    for i in (0, heads // 2, heads - 1):
        rows = ix[off[i]:off[i + 1]]
        lt = _want(K, V, i, r, dtype, "kv", True)
        gu.check_scores(sc[i].cpu().numpy(), lt, str(i))
        gu.check_selection(rows.cpu().numpy().astype(np.int64), lt, int(budgets[i]), 4, str(i))
        assert torch.equal(Ko[off[i]:off[i + 1]], K[i][rows.long()]) and torch.equal(Vo[off[i]:off[i + 1]], V[i][rows.long()])


# Budgets around what counts as even (the largest a quarter above the average), gathered by the selection kernel: rows past the caches from the lower limit
# on where they are, with the heads along the grid's x, and from the upper one on where they are not, with the shares along x.  fp32 over the bf16 units both ways
@pytest.mark.parametrize("heads,n,dtype", [(64, 6103, "bf16"), (64, 7900, "bf16"), (32, 9700, "bf16"), (112, 1744, "fp32"), (64, 4090, "fp32")])
@pytest.mark.parametrize("more", [0, 1])
def test_one_call_at_the_edge_of_even_budgets(heads, n, dtype, more):
    import torch
    average, s = 400, 4
    bytes_read = heads * n * 128 * (2 if dtype == "bf16" else 4) * 2
    K, V = _cache(heads, n, dtype, n)
    budgets = np.full((heads,), average, np.int32)
    budgets[3] += average // 4 + more
    budgets[9] -= average // 4 + more
    even = int(budgets.max()) * heads * 4 <= int(budgets.sum()) * 5
    assert even == (more == 0)
    with B.Context(heads, 1, 4, 128, 20, dtype, n, SEED) as ctx:
        sc, ix, Ko, Vo, off = gu.run_path(ctx, K, V, n, budgets, s, dtype, one_call=True)
        scan, select = gu.launches(lambda: ctx.compress(K, V, n, budgets, s, off, sc, ix, Ko, Vo))
    past = bytes_read > (LIMIT_REREAD if even else LIMIT_REREAD_MANY)
    assert scan[:2] == (("scores_bf16_kernel", (2, 0, 1, 0, int(past))) if dtype == "bf16" else ("scores_f32_kernel", (2, 0, 1, 0, 1, int(bytes_read > LIMIT_REREAD_MANY))))
    assert select[0] == "select_gather_kernel"
    if n > 2048:
        assert (select[2][0] == heads) == even
    for i in (0, 3, 9, heads - 1):
        rows = ix[off[i]:off[i + 1]]
        lt = _want(K, V, i, 20, dtype, "kv", True)
        gu.check_scores(sc[i].cpu().numpy(), lt, str(i))
        gu.check_selection(rows.cpu().numpy().astype(np.int64), lt, int(budgets[i]), s, str(i))
        assert torch.equal(Ko[off[i]:off[i + 1]], K[i][rows.long()]) and torch.equal(Vo[off[i]:off[i + 1]], V[i][rows.long()])


FUSED_MANY = gu.limit("fused_kernel.hip", "kFusedStreamBytesMany")


# one tensor scored, one workgroup a head: few rows kept are streamed from 2049 tokens on, a quarter and more from a number of bytes on; gathered by the
# same kernel, by kernels of their own, and after budgets allotted on the device
@pytest.mark.parametrize("source,r,projection", [("k", 64, True), ("v", 20, True), ("v", 64, False)])
@pytest.mark.parametrize("tokens,keep", [("first", 0.1), ("first", 0.3), ("first", 0.5), ("last", 0.5), ("more", 0.5)])
def test_one_tensor_by_one_workgroup_a_head(source, r, projection, tokens, keep):
    import torch
    heads, s = torch.cuda.get_device_properties(0).multi_processor_count, 4
    last = FUSED_MANY // (heads * 256)
    n = {"first": 2049, "last": last, "more": last + 1}[tokens]
    K, V = _cache(heads, n, "bf16", n + r)
    budgets = np.full((heads,), int(np.ceil(keep * n)), np.int32)
    with B.Context(heads, 1, 4, 128, r, "bf16", n, SEED, source, projection) as ctx:
        sc, ix, Ko, Vo, off = gu.run_path(ctx, K, V, n, budgets, s, "bf16", one_call=True)
        scan = gu.launches(lambda: ctx.compress(K, V, n, budgets, s, off, sc, ix, Ko, Vo))[0]
        torch.cuda.synchronize()
        args = (4 if r > 32 and projection else 2, 8, 1 if source == "k" else 2, int(projection), 2 if keep < 0.25 or tokens == "more" else 0)
        assert scan[:2] == ("fused_kernel", args), scan
        bo, oo = torch.empty((heads,), dtype=torch.int32, device="cuda"), torch.empty((heads + 1,), dtype=torch.int64, device="cuda")
        sc2, ix2, Ko2, Vo2 = torch.full_like(sc, float("nan")), torch.empty_like(ix), torch.empty_like(Ko), torch.empty_like(Vo)
        call = lambda: ctx.compress_adaptive(K, V, n, int(budgets[0]), s, 0.2, sc2, bo, oo, ix2, Ko2, Vo2)
        call()
        assert gu.launches(call)[0][:2] == scan[:2]
        torch.cuda.synchronize()
    assert torch.equal(sc, sc2) and torch.equal(ix, ix2) and torch.equal(Ko, Ko2) and torch.equal(Vo, Vo2)      # (one head a layer: its budget is the layer's)
    for i in (0, heads // 2, heads - 1):
        rows = ix[off[i]:off[i + 1]]
        lt = _want(K, V, i, r, "bf16", source, projection)
        gu.check_scores(sc[i].cpu().numpy(), lt, str(i))
        gu.check_selection(rows.cpu().numpy().astype(np.int64), lt, int(budgets[i]), s, str(i))
        assert torch.equal(Ko[off[i]:off[i + 1]], K[i][rows.long()]) and torch.equal(Vo[off[i]:off[i + 1]], V[i][rows.long()])


START = gu.limit("scores_kernels.hip", "kStartHeadBytes")


# one workgroup takes long over a head: the start of its scan goes through the caches, from a number of bytes a head on, then the rows go past them, and at the end through them again
# where many are kept; by the kernel that does everything, by it and separate kernels, and by the general ones, which take several workgroups a head instead up to four fifths of the units
@pytest.mark.parametrize("heads,r,keep,dtype,source", [(256, 64, 0.05, "bf16", "kv"), (256, 20, 0.5, "bf16", "kv"), (205, 20, 0.1, "bf16", "kv"), (205, 64, 0.4, "bf16", "kv"), (204, 20, 0.1, "bf16", "kv"), (192, 64, 0.4, "bf16", "kv"), (256, 128, 0.1, "bf16", "kv"),
                                                       (256, 20, 0.1, "fp32", "kv"), (256, 32, 0.4, "fp32", "kv")])
@pytest.mark.parametrize("side", ["below", "from"])
def test_the_start_of_a_long_scan(heads, r, keep, dtype, source, side):
    import torch
    units = torch.cuda.get_device_properties(0).multi_processor_count
    heads, s = heads * units // 256, 4
    row = 128 * (2 if dtype == "bf16" else 4) * (2 if source == "kv" else 1)
    n = (START - 1) // row + (side == "from")
    assert (n * row >= START) == (side == "from")
    K, V = _cache(heads, n, dtype, n + r)
    budgets = np.full((heads,), int(keep * n), np.int32)
    with B.Context(heads, 1, 4, 128, r, dtype, n, SEED, source) as ctx:
        sc, ix, Ko, Vo, off = gu.run_path(ctx, K, V, n, budgets, s, dtype, one_call=True)
        name, args, grid = gu.launches(lambda: ctx.compress(K, V, n, budgets, s, off, sc, ix, Ko, Vo))[0]
        torch.cuda.synchronize()
    one = side == "below" or heads * 5 >= units * 4             # one workgroup a head
    assert (grid[0] == heads) == one, (name, grid)
    if name == "scores_bf16_kernel":
        assert args[4] == (2 if (side == "from" and one) or keep >= 0.25 else 1), args
    else:
        assert name == ("fused_kernel" if dtype == "bf16" else "scores_f32_kernel") and args[4:] == ((2,) if dtype == "bf16" else (1, 1)), (name, args)
    for i in (0, heads // 2, heads - 1):
        rows = ix[off[i]:off[i + 1]]
        lt = _want(K, V, i, r, dtype, source, True)
        gu.check_scores(sc[i].cpu().numpy(), lt, str(i))
        assert np.linalg.norm(sc[i].cpu().numpy() - lt) <= NORM_TOL * np.linalg.norm(lt), i
        gu.check_selection(rows.cpu().numpy().astype(np.int64), lt, int(budgets[i]), s, str(i))
        assert torch.equal(Ko[off[i]:off[i + 1]], K[i][rows.long()]) and torch.equal(Vo[off[i]:off[i + 1]], V[i][rows.long()])


# up to 32 columns of an fp32 cache: rows of a call that gathers stay in the caches up to a number of bytes; gathered by the selection, by the split selection that has its counts
# from the scoring and by a kernel of its own, one tensor scored and both, to whole and ragged groups
@pytest.mark.parametrize("heads,n,r,source,keep", [(128, 1024, 20, "kv", 0.1), (8, 24000, 32, "kv", 0.2), (8, 24011, 20, "k", 0.1), (16, 16301, 20, "v", 0.2), (3, 65001, 32, "kv", 0.1), (5, 60001, 20, "k", 0.4),
                                                   (100, 2099, 20, "kv", 0.7), (256, 1009, 20, "v", 0.1)])
def test_one_call_of_narrow_sketches_in_fp32(heads, n, r, source, keep):
    import torch
    bytes_read, s = heads * n * 512 * (2 if source == "kv" else 1), 4
    assert bytes_read <= LIMIT_REREAD_MANY
    K, V = _cache(heads, n, "fp32", n + r)
    budgets = np.full((heads,), int(keep * n), np.int32)
    with B.Context(heads, 1, 4, 128, r, "fp32", n, SEED, source) as ctx:
        sc, ix, Ko, Vo, off = gu.run_path(ctx, K, V, n, budgets, s, "fp32", one_call=True)
        name, args, _ = gu.launches(lambda: ctx.compress(K, V, n, budgets, s, off, sc, ix, Ko, Vo))[0]
        torch.cuda.synchronize()
    assert (name, args) == ("scores_f32_kernel", (2, {"kv": 0, "k": 1, "v": 2}[source], 1, int(n > 24576), 1, 0)), (name, args)
    for i in (0, heads // 2, heads - 1):
        rows = ix[off[i]:off[i + 1]]
        lt = _want(K, V, i, r, "fp32", source, True)
        gu.check_scores(sc[i].cpu().numpy(), lt, str(i))
        assert np.linalg.norm(sc[i].cpu().numpy() - lt) <= NORM_TOL * np.linalg.norm(lt), i
        gu.check_selection(rows.cpu().numpy().astype(np.int64), lt, int(budgets[i]), s, str(i))
        assert torch.equal(Ko[off[i]:off[i + 1]], K[i][rows.long()]) and torch.equal(Vo[off[i]:off[i + 1]], V[i][rows.long()])
