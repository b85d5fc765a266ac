"""The selection of long heads by several workgroups per head: against the oracle's selection on the very
scores the library stored, so that every index has to agree, ties included."""
import numpy as np
import pytest

from oracle import curdkv_oracle as orc
from paper_2509_15038_amd import binding as B
from paper_2509_15038_amd import workloads as wl
from tests import gpu_util as gu

pytestmark = pytest.mark.gpu


def _check(scores, idx, off, budgets, s):
    for i, k in enumerate(budgets):
        want = orc.select(scores[i].astype(np.float64), int(k), s)
        assert np.array_equal(idx[off[i]:off[i + 1]], want), (i, int(k), s)


def _select(scores, budgets, s):
    import torch
    heads, n = scores.shape
    off = wl.offsets_for(budgets)
    with B.Context(1, heads, 4, 128, 32, "bf16", n, 1) as ctx:
        g = gu.Guarded((max(int(off[-1]), 1),), torch.int32, -7)
        ctx.select(torch.from_numpy(scores).cuda(), n, budgets, s, off, g.t)
        torch.cuda.synchronize()
        g.check("indices")
        return g.t.cpu().numpy().astype(np.int64), off


# (36864: the longest head one workgroup takes; 131072: the longest the bitmaps take)
@pytest.mark.parametrize("n", [36864, 36865, 40960, 65537, 131071, 131072, 131073])
def test_given_scores(n):
    rng = np.random.default_rng(n)
    x = np.exp(rng.standard_normal((9, n)) * 2.0)
    x[1] = 1.0                                                # one value: every candidate ties
    x[2] = rng.integers(0, 3, n)                              # three values, zero among them
    x[3] = np.round(rng.random(n) * 7000) + 1                 # ties everywhere
    x[4] = 1.0 + rng.random(n) * 1e-3                         # one bin holds the whole head
    x[5] *= 1e-33                                             # normalised scores below 1e-37 among them
    x[6, : n // 2] = 0.0
    x[7] = rng.random(n) * 3.0                                # (not normalised below: scores of 2 and above)
    x[8, n - 5:] = 1e6                                        # a block at the end
    norm = x.sum(1, keepdims=True)
    norm[7] = 1.0
    scores = (x / norm).astype(np.float32)
    for budgets, s in ((np.array([n // 10] * 9), 4), (np.array([0, 1, 4, 5, n - 1, n, n // 2, n // 3, 6]), 4),
                       (np.array([n // 2] * 9), 0), (np.array([70, n - 64, 130, 4096, 4097, 64, 65, 1, n]), 64)):
        budgets = budgets.astype(np.int32)
        idx, off = _select(scores, budgets, s)
        _check(scores, idx, off, budgets, s)


PAIRS, LIST = gu.limit("split_select.hip", "kSplitPairs"), gu.limit("split_select.hip", "kSplitList")


# keys that share the cut's bin [1, 1 + 1/16): as many as are resolved in LDS, in registers, and by reading the scores
# again, and one more; tokens on both sides of 65536 or not
@pytest.mark.parametrize("n", [50000, 131072])
@pytest.mark.parametrize("inside", [1, 511, PAIRS, PAIRS + 1, 8192, LIST, LIST + 1, 40000])
def test_range_of_every_size(n, inside):
    rng = np.random.Generator(np.random.PCG64([n, inside]))
    above, heads = 300, 8
    scores = rng.uniform(0.0, 0.5, (heads, n)).astype(np.float32)
    budgets = np.zeros((heads,), np.int32)
    for h in range(heads):
        place = rng.permutation(np.arange(4, n))
        scores[h, place[:above]] = rng.uniform(1.5, 1.9, above)
        fine = (1.0 + rng.integers(0, 2 ** 19, inside) * 2.0 ** -23).astype(np.float32)
        if h in (2, 3):                                       # half of them from eight values
            fine = np.where(rng.random(inside) < 0.5, 1.0 + rng.integers(0, 8, inside) / 128.0, fine)
        if h in (4, 5):                                       # three neighbouring floats, at the end of the bin
            fine = 1.0625 - (1 + rng.integers(0, 3, inside)) * 2.0 ** -23
        if h == 6:                                            # one value
            fine = 1.03125
        scores[h, place[above:above + inside]] = fine
        if h == 7:                                            # all in one stretch
            scores[h, 4:] = np.concatenate([scores[h, place[above:above + inside]], np.delete(scores[h], place[above:above + inside])[4:]])
        budgets[h] = 4 + above + (1, inside, (inside + 1) // 2, inside // 3 + 1, (inside + 1) // 2, inside // 5 + 1, inside // 2 + 1, inside // 7 + 1)[h]
    idx, off = _select(scores, budgets, 4)
    _check(scores, idx, off, budgets, 4)


def _one_call(K, V, dtype, r, budgets, s, with_scores=True, sketch=None):
    import torch
    L, H, n, d = K.shape
    off = wl.offsets_for(budgets)
    tdt = torch.bfloat16 if dtype == "bf16" else torch.float32
    total = int(off[-1])
    with B.Context(L, H, 4, d, r, dtype, n, 7) as ctx:
        for h in range(H if sketch is not None else 0):
            ctx.set_sketch(0, h, sketch)
        Kd, Vd = gu.to_device(K, dtype), gu.to_device(V, dtype)
        sc = gu.Guarded((L * H, n), torch.float32, float("nan"))
        ix = gu.Guarded((max(total, 1),), torch.int32, -7)
        Ko = gu.Guarded((max(total, 1), d), tdt, float("nan"))
        Vo = gu.Guarded((max(total, 1), d), tdt, float("nan"))
        ctx.compress(Kd, Vd, n, budgets, s, off, sc.t if with_scores else None, ix.t, Ko.t, Vo.t)
        torch.cuda.synchronize()
        for g in (sc, ix, Ko, Vo):
            g.check()
        idx = ix.t.cpu().numpy().astype(np.int64)[:total]
        ko, vo = gu.to_host(Ko.t, dtype)[:total], gu.to_host(Vo.t, dtype)[:total]
        for i in range(L * H):
            rows = idx[off[i]:off[i + 1]]
            assert np.array_equal(ko[off[i]:off[i + 1]], K.reshape(L * H, n, d)[i][rows])
            assert np.array_equal(vo[off[i]:off[i + 1]], V.reshape(L * H, n, d)[i][rows])
        return sc.t.cpu().numpy(), idx, off


# 1 to 33 heads on both sides of the lengths at which the route changes (up to 32768 tokens, with few rows, it is the selection that gathers
# as well); 128 columns and fp32 have other scoring kernels
@pytest.mark.parametrize("heads,n,r,dtype", [(1, 24576, 20, "bf16"), (1, 24577, 20, "bf16"), (3, 30001, 64, "bf16"), (33, 36865, 20, "bf16"),
                                             (1, 32768, 20, "bf16"), (1, 32769, 20, "bf16"), (3, 33001, 64, "bf16"), (8, 32767, 20, "bf16"),
                                             (2, 131072, 128, "bf16"), (1, 50000, 20, "fp32"), (2, 33333, 64, "fp32"), (1, 40000, 128, "fp32")])
def test_one_call(heads, n, r, dtype):
    cfg = wl.scaled(wl.CONFIGS["c2"], kv_heads=heads, n=n, r=r, dtype=dtype)
    K, V = wl.host_cache(cfg)
    if heads > 1:                                             # a head of few distinct rows: ties by the thousand, also at the bins' ends
        few = np.random.default_rng(1).integers(0, 40, n)
        K[0, 1], V[0, 1] = K[0, 1][few], V[0, 1][few]
    if heads > 2:
        V[0, 2] = 0                                           # a head of zeros: uniform scores
    budgets = np.array([n // 10, n // 3, n // 2, 0, 3, n, n - 1, 64][:heads] + [n // 7] * max(0, heads - 8), dtype=np.int32)
    scores, idx, off = _one_call(K, V, dtype, r, budgets, 4)
    assert np.all(np.isfinite(scores))
    _check(scores, idx, off, budgets, 4)
    _, idx2, _ = _one_call(K, V, dtype, r, budgets, 4, with_scores=False)
    assert np.array_equal(idx, idx2)


# (counted in the scan: more than two heads, and longer ones than the selection that gathers takes)
@pytest.mark.parametrize("r,n", [(64, 33002), (128, 33002), (64, 30002)])
def test_rows_scored_again(r, n):
    """fp32 rows whose split into bf16 parts overflows (a float above the largest bf16, in a dimension that
    the sketch leaves out) but whose score is finite: counted once, in the bin of that score."""
    s = 4
    cfg = wl.scaled(wl.CONFIGS["c2"], kv_heads=6, n=n, r=r, dtype="fp32")
    K, V = wl.host_cache(cfg)
    rng = np.random.default_rng(r)
    G = (rng.standard_normal((128, r)) / np.sqrt(r)).astype(np.float32)
    G[[9, 100]] = 0.0
    for h in range(6):
        rows = rng.permutation(n)[:(0, 1, 300, 300, 300, 3000)[h]]
        (K if h % 2 else V)[0, h, rows, 9] = np.finfo(np.float32).max
        K[0, h, rows[::3], 100] = -np.finfo(np.float32).max
        K[0, h, 2, 9] = np.finfo(np.float32).max              # a sink: counted nowhere
    for frac in (7, 40, 1000):
        budgets = np.array([s + 1, n // frac, s + 1, s + 2, n // frac, n // frac], dtype=np.int32)
        scores, idx, off = _one_call(K, V, "fp32", r, budgets, s, sketch=G)
        _check(scores, idx, off, budgets, s)
    for h in range(6):
        want = orc.scores(K[0, h].astype(np.float64), V[0, h].astype(np.float64), G.astype(np.float64), "kv")
        gu.check_scores(scores[h], want, h)


def test_scores_out_of_the_ordinary():
    """Scores that curdkv_scores itself can leave (an infinite product gives NaN), and zeros of either sign, keep the
    same tokens as in a context of more heads than this route takes; scores that have no business
    here (negative ones) have no order, but keep as many tokens as asked for."""
    n, s, most = 40001, 4, gu.limit("curdkv_internal.h", "kSplitMaxHeads")
    rng = np.random.default_rng(9)
    x = np.exp(rng.standard_normal((most + 1, n)) * 2.0).astype(np.float32)
    x[0, rng.permutation(n)[:50]] = np.nan
    x[1, rng.permutation(n)[:50]] = np.inf
    x[2, ::2] = -0.0
    x[3] *= np.where(rng.random(n) < 0.3, -1, 1)
    x[4, ::3] = -np.float32(np.nan)
    x[5] = -x[5]
    budgets = np.full((most + 1,), 9, np.int32)
    for k in (5, 30, 60, n // 3, n - 1):
        budgets[:6] = k
        want, off = _select(x, budgets, s)                    # one workgroup per head
        got, off6 = _select(np.ascontiguousarray(x[:6]), budgets[:6].copy(), s)
        assert np.array_equal(got[:off[3]], want[:off[3]])
        assert got.min() == 0 and got.max() < n and np.all(np.diff(got.reshape(6, k)) > 0)


# the selection that gathers, the split one, one workgroup per head, a head in parts, the fused kernel; and the two separate normalisations
@pytest.mark.parametrize("heads,n,dtype", [(2, 30001, "fp32"), (2, 33001, "fp32"), (33, 30001, "bf16"), (33, 34001, "bf16"), (129, 37001, "bf16"), (256, 700, "bf16"), (2, 300, "fp32")])
def test_sum_too_small_to_divide_by(heads, n, dtype):
    """A head whose scores add up to less than the smallest number with a finite reciprocal (2.9e-39) keeps
    finite scores, in their order."""
    import torch
    s = 4
    K = torch.zeros((heads, n, 128), dtype=torch.bfloat16 if dtype == "bf16" else torch.float32, device="cuda")
    V = torch.zeros_like(K)
    g = torch.Generator(device="cuda")
    g.manual_seed(5)
    rows = torch.randperm(n, generator=g, device="cuda")[:100].sort().values
    K[:2, rows] = 1e-11
    V[:2, rows] = (2e-13 * (1 + torch.arange(100, device="cuda") % 7)[:, None]).to(V.dtype)
    with B.Context(1, heads, 4, 128, 20, dtype, n, 7) as ctx:
        sc = torch.empty((heads, n), device="cuda")
        Ko, Vo = torch.empty((2 * n, 128), dtype=K.dtype, device="cuda"), torch.empty((2 * n, 128), dtype=K.dtype, device="cuda")
        for k in (5, 60, 104, n // 2, n - 1):
            budgets = np.array([k, k] + [0] * (heads - 2), np.int32)
            off = wl.offsets_for(budgets)
            ix = torch.full((2 * k,), -7, dtype=torch.int32, device="cuda")
            ctx.compress(K, V, n, budgets, s, off, sc, ix, Ko, Vo)
            got = sc[:2].cpu().numpy()
            assert np.all(np.isfinite(got)) and np.count_nonzero(got) == 200 and len(np.unique(got[0])) > 4
            _check(got, ix.cpu().numpy(), off, budgets[:2], s)
        raw, sums, two = torch.empty_like(sc), torch.zeros((heads,), dtype=torch.float64, device="cuda"), torch.empty_like(sc)
        ctx.scores_append(K, V, n, 0, n, raw, sums)
        assert 0 < float(sums[0]) < 2.9e-39
        ctx.normalise(raw, sums, n, n, two)
        ctx.scores(K, V, n, sc)
        for x in (two, sc):
            assert bool(torch.isfinite(x[:2]).all()) and int(torch.count_nonzero(x[:2])) == 200


# the heads along the grid's x where the budgets are even, the largest at most a quarter above the average; lists alone, and with the rows
@pytest.mark.parametrize("more", [0, 1])
@pytest.mark.parametrize("one_call", [False, True])
def test_order_of_the_grid(more, one_call):
    import torch
    heads, n, average = 6, 40000, 4000
    budgets = np.full((heads,), average, np.int32)
    budgets[2] += average // 4 + more
    budgets[3] -= average // 4 + more
    g = torch.Generator(device="cuda")
    g.manual_seed(more)
    K, V = (torch.randn((1, heads, n, 128), generator=g, device="cuda").to(torch.bfloat16) for _ in range(2))
    with B.Context(1, heads, 4, 128, 20, "bf16", n, 3) as ctx:
        sc, idx, Ko, Vo, off = gu.run_path(ctx, K, V, n, budgets, 4, "bf16", one_call=one_call)
        call = (lambda: ctx.compress(K, V, n, budgets, 4, off, sc, idx, Ko, Vo)) if one_call else (lambda: ctx.select(sc, n, budgets, 4, off, idx))
        name, args, grid = gu.launches(call)[-1]
        torch.cuda.synchronize()
    assert name == "split_emit_kernel" and args[0] == (16 if one_call else 0) and (grid[0] == heads) == (more == 0) and heads in grid, (name, args, grid)
    where = idx.long()
    for h in range(heads):
        mine = slice(int(off[h]), int(off[h + 1]))
        assert np.array_equal(where[mine].cpu().numpy(), orc.select(sc[h].cpu().numpy().astype(np.float64), int(budgets[h]), 4)), h
        assert torch.equal(Ko[mine], K[0, h, where[mine]]) and torch.equal(Vo[mine], V[0, h, where[mine]]), h
