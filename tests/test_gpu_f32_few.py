"""fp32 calls of few tokens in all: workgroups of 16 tokens whose waves share the products.  Scores
and running sums against the float64 oracle at the edges of the 16-token steps, with one step and
several per workgroup, around the lines where the other kernels take over, and the
other kernels on rows that are not finite at a size that is theirs."""
import numpy as np
import pytest

from oracle import curdkv_oracle as orc
from paper_2509_15038_amd import binding as B
from paper_2509_15038_amd import workloads as wl

pytestmark = pytest.mark.gpu

SEED = 0xC0DE0009
# a projected coordinate is 128 products rounded once per 4 (32 roundings of 2^-24, at random), squared
# and summed over r, multiplied and normalised: the same terms as for the wider calls
NORM_TOL = 1e-6


# one token; edges of a step; 64 workgroups of 1, 2 and 6 steps (the last ones short or empty), and one step more; many heads, around the tokens up to which
# every width is taken (beyond them, (65, 256) and (2049, 8), r = 20 is by its load, and the wider ones are not: test_gpu_few_load.py asks which kernel runs)
@pytest.mark.parametrize("n,heads", [(1, 1), (16, 1), (17, 3), (1024, 1), (1025, 1), (6144, 1), (6145, 1),
                                     (1, 256), (33, 256), (64, 256), (65, 256), (2048, 8), (2049, 8)])
@pytest.mark.parametrize("r,source", [(20, "kv"), (33, "kv"), (64, "k"), (128, "kv"), (128, "v")])
def test_scores_and_sums(n, heads, r, source):
    import torch
    cfg = wl.scaled(wl.CONFIGS["c2"], layers=heads, kv_heads=1, n=n, r=r, dtype="fp32")
    K, V = wl.host_cache(cfg)
    dK, dV = torch.from_numpy(K).cuda(), torch.from_numpy(V).cuda()
    with B.Context(heads, 1, 4, 128, r, "fp32", n + 7, SEED, source) as ctx:
        got = torch.full((heads, n), float("nan"), device="cuda")
        ctx.scores(dK, dV, n, got)
        # behind five tokens scored before, in rows of n + 7 places: only the new ones are written
        raw = torch.full((heads, n + 7), -1.0, device="cuda")
        sums = torch.full((heads,), 3.0, dtype=torch.float64, device="cuda")
        ctx.scores_append(dK, dV, n, 5, n + 7, raw, sums)
        got, raw, sums = got.cpu().numpy(), raw.cpu().numpy(), sums.cpu().numpy()
    assert np.all(raw[:, :5] == -1.0) and np.all(raw[:, n + 5:] == -1.0)
    assert np.allclose(sums - 3.0, raw[:, 5:n + 5].astype(np.float64).sum(1), rtol=1e-6)
    for i in range(heads) if heads < 8 else (0, heads // 2, heads - 1):
        G = orc.sketch(SEED, i, 0, 1, 128, r, "fp32")
        want = orc.scores(K[i, 0].astype(np.float64), V[i, 0].astype(np.float64), G, source)
        assert np.linalg.norm(got[i] - want) <= NORM_TOL * np.linalg.norm(want), (n, heads, r, source, i)
        new = raw[i, 5:n + 5].astype(np.float64)
        assert np.linalg.norm(new / new.sum() - want) <= NORM_TOL * np.linalg.norm(want)


@pytest.mark.parametrize("n,layers", [(300, 1), (300, 64)])     # this kernel, and the split products
@pytest.mark.parametrize("r", [64, 128])
def test_rows_that_are_not_finite(n, layers, r):
    import torch
    cfg = wl.scaled(wl.CONFIGS["c2"], layers=layers, kv_heads=1, n=n, r=r, dtype="fp32")
    K, V = wl.host_cache(cfg)

    def raw_scores():
        with B.Context(layers, 1, 4, 128, r, "fp32", n, SEED) as ctx:
            raw = torch.full((layers, n), -1.0, device="cuda")
            sums = torch.zeros((layers,), dtype=torch.float64, device="cuda")
            ctx.scores_append(torch.from_numpy(K).cuda(), torch.from_numpy(V).cuda(), n, 0, n, raw, sums)
            return raw.cpu().numpy()

    clean = raw_scores()
    K[0, 0, 5, 17] = np.inf
    K[0, 0, 130, 3] = np.finfo(np.float32).max
    V[0, 0, 77, 100] = np.nan
    V[0, 0, 299, 0] = -np.inf
    raw = raw_scores()
    assert np.all(np.isposinf(raw[0, [5, 130, 299]])) and np.isnan(raw[0, 77])
    rest = np.setdiff1d(np.arange(n), [5, 77, 130, 299])
    assert np.array_equal(raw[0, rest], clean[0, rest]) and np.array_equal(raw[1:], clean[1:])
