"""fp32 caches with more than 32 sketch columns: every float goes through the bf16 matrix units as
three bf16 numbers.  Scores against the float64 oracle, and rows that are not finite.  (Calls of few tokens in all,
the smaller sizes here, take a kernel of plain fp32 products; the edges of this one's steps, groups and
ranges beyond that limit are in test_gpu_dispatch_sides.py.)"""
import numpy as np
import pytest

from oracle import curdkv_oracle as orc
from paper_2509_15038_amd import binding as B
from paper_2509_15038_amd import workloads as wl

pytestmark = pytest.mark.gpu

# 2-norm error of a head's scores: a projected coordinate is 128 exact products, summed with one
# rounding per 32 of them over six passes (24 roundings), the parts left out weigh 2^-24 of a product at most
# and 2^-27 at root mean square; squared and summed over r, multiplied and normalised (about 30 roundings
# of 2^-24 relative, at random)
NORM_TOL = 1e-6


def _scores(K, V, r, source, seed=0xC0DE0009):
    import torch
    L, H, n, d = K.shape
    with B.Context(L, H, 4, d, r, "fp32", n, seed, source) as ctx:
        out = torch.full((L * H, n), float("nan"), device="cuda")
        ctx.scores(torch.from_numpy(K).cuda(), torch.from_numpy(V).cuda(), n, out)
        raw = torch.full((L * H, n), float("nan"), device="cuda")
        sums = torch.zeros((L * H,), dtype=torch.float64, device="cuda")
        ctx.scores_append(torch.from_numpy(K).cuda(), torch.from_numpy(V).cuda(), n, 0, n, raw, sums)
        return out.cpu().numpy(), raw.cpu().numpy()


# (the last: 9 workgroups' waves with ranges of several groups, the last one short)
@pytest.mark.parametrize("n,layers", [(1, 1), (15, 1), (17, 2), (64, 1), (65, 2), (1009, 1), (2048 + 37, 64)])
@pytest.mark.parametrize("r,source", [(33, "kv"), (64, "k"), (64, "kv"), (65, "v"), (128, "kv")])
def test_scores_against_the_oracle(n, layers, r, source):
    cfg = wl.scaled(wl.CONFIGS["c2"], layers=layers, kv_heads=2, n=n, r=r, dtype="fp32")
    K, V = wl.host_cache(cfg)
    got, _ = _scores(K, V, r, source)
    for i in range(layers * 2) if layers < 8 else (0, 5, layers * 2 - 1):
        G = orc.sketch(0xC0DE0009, i // 2, i % 2, 2, 128, r, "fp32")
        want = orc.scores(K[i // 2, i % 2].astype(np.float64), V[i // 2, i % 2].astype(np.float64), G, source)
        assert np.linalg.norm(got[i] - want) <= NORM_TOL * np.linalg.norm(want), (n, r, source, i)


@pytest.mark.parametrize("r", [64, 128])
def test_rows_that_are_not_finite(r):
    """A row with an infinity, one at the top of the fp32 range (its bf16 rounding is infinite) and one
    with a NaN score what plain fp32 arithmetic gives them; every other row is as without them."""
    cfg = wl.scaled(wl.CONFIGS["c2"], layers=1, kv_heads=1, n=300, r=r, dtype="fp32")
    K, V = wl.host_cache(cfg)
    _, clean = _scores(K, V, r, "kv")
    K[0, 0, 5, 17] = np.inf
    K[0, 0, 130, 3] = np.finfo(np.float32).max
    V[0, 0, 77, 100] = np.nan
    V[0, 0, 299, 0] = -np.inf
    _, raw = _scores(K, V, r, "kv")
    assert np.all(np.isposinf(raw[0, [5, 130, 299]])) and np.isnan(raw[0, 77])
    rest = np.setdiff1d(np.arange(300), [5, 77, 130, 299])
    assert np.array_equal(raw[0, rest], clean[0, rest])
