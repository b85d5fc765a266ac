"""fp32 caches with more than 32 sketch columns, and with fewer from a number of tokens on: every float goes through the bf16 matrix units as
three bf16 numbers.  Scores against the float64 oracle, and rows that are not finite.  (Calls of few tokens in all,
the smaller sizes here, take a kernel of plain fp32 products; the edges of this one's steps, groups and
ranges beyond that limit are in test_gpu_dispatch_sides.py.)"""
import numpy as np
import pytest

from oracle import curdkv_oracle as orc
from paper_2509_15038_amd import binding as B
from paper_2509_15038_amd import workloads as wl
from tests import gpu_util as gu

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


# The error of one score: a projected coordinate errs by some 24 roundings of its running sum, 1.5e-7 at root mean square, a
# norm of 33 such coordinates by 5e-8, a score by 9e-8 with its squares and the last rounding; five times that over the 30000 scores compared, and twice
# that again for rows that lean on few coordinates.
ELEMENT_TOL = 16 * 2.0 ** -24


# (20 and 32 columns: fewer coordinates to a norm, so 1.2e-7 to a score, and 190000 scores compared; 64 heads of 3001 tokens are split there)
@pytest.mark.parametrize("r", [20, 32, 33, 64, 128])
@pytest.mark.parametrize("rows", ["scaled", "uncovered", "zero sketch", "unlike 8", "unlike 12", "unlike 14", "unlike 20", "white 2", "white 3"])
def test_rows_and_sketches_of_any_size(r, rows):
    """Rows between 1e-8 and 1e8 (products of squared norms stay below 2^127); a sketch that is zero where the rows are
    largest; a sketch of zeros, and rows of zeros; sketches that make up for channels of unlike size: 40 channels 2^p times the
    others, or log-normal ones, and the rows of the sketch as much smaller, so that every element matters alike."""
    import torch
    L, H, n = (2, 8, 2048 + 37) if r > 32 else (8, 8, 3001)            # beyond the calls of few tokens, and of plain products
    tol = ELEMENT_TOL if r > 32 else 1.5 * ELEMENT_TOL
    rng = np.random.default_rng([5, r])
    K, V = (rng.standard_normal((L, H, n, 128)).astype(np.float32) for _ in range(2))
    G = (rng.standard_normal((128, r)) / np.sqrt(r)).astype(np.float32)
    if rows == "scaled":
        K *= np.exp(rng.uniform(-18, 18, (L, H, n, 1))).astype(np.float32)
        V *= np.exp(rng.uniform(-18, 18, (L, H, n, 1))).astype(np.float32)
    elif rows == "uncovered":
        G[:40] = 0
        K[..., :40] *= 1e8
        V[..., 7] *= np.exp(rng.uniform(0, 30, (L, H, n))).astype(np.float32)
    elif rows == "zero sketch":
        G[:] = 0
    else:
        kind, p = rows.split()
        size = np.where(np.arange(128) < 40, 2.0 ** int(p), 1.0) if kind == "unlike" else np.exp(rng.standard_normal(128) * int(p))
        K, V, G = (K * size).astype(np.float32), (V * size).astype(np.float32), (G / size[:, None]).astype(np.float32)
    K[1, 3, 99:140] = 0
    K[0, 0, 130, 50], V[0, 0, 77, 100], V[0, 0, 2084, 0], K[0, 0, 64, 64] = np.inf, np.nan, -np.inf, np.finfo(np.float32).max
    with B.Context(L, H, 4, 128, r, "fp32", n, 1) as ctx:
        for i in range(L * H):
            ctx.set_sketch(i // H, i % H, G)
        raw = torch.full((L * H, n), float("nan"), device="cuda")
        sums = torch.zeros((L * H,), dtype=torch.float64, device="cuda")
        dK, dV = torch.from_numpy(K).cuda(), torch.from_numpy(V).cuda()
        ctx.scores_append(dK, dV, n, 0, n, raw, sums)
        name, args, _ = gu.launches(lambda: ctx.scores_append(dK, dV, n, 0, n, raw, sums))[0]
        assert name == "scores_f32_kernel" and args[4] == 1, (name, args)
        raw = raw.cpu().numpy().reshape(L, H, n)
    for i, j in np.ndindex(L, H):
        K64, V64, G64 = (x.astype(np.float64) for x in (K[i, j], V[i, j], G))
        with np.errstate(invalid="ignore"):
            want = ((K64 @ G64) ** 2).sum(1) * ((V64 @ G64) ** 2).sum(1)
        if (i, j) == (0, 0):
            if rows == "scaled":                                        # (in some others infinities meet zeros of the sketch, at r = 33 of its padding)
                assert np.isnan(raw[0, 0, 77]) and np.all(np.isposinf(raw[0, 0, [64, 130, 2084] if r not in (20, 33) else [64]]))
            raw[0, 0, [64, 77, 130, 2084]] = want[[64, 77, 130, 2084]] = 0
        assert np.all(np.abs(raw[i, j] - want) <= tol * want), (i, j)


# Plain fp32 products round a coordinate's sum once per 4 of them, 32 times instead of 24 of a finer sum: a score of 20 to 32 columns errs by
# 2e-7 at root mean square, seven times that over the 130000 scores compared, and twice that again for rows that lean on few coordinates ("largest": on one).
PLAIN_TOL = 48 * 2.0 ** -24


# Up to 32 columns the split products are taken from a number of tokens on only: what plain fp32 products give for a caller's own sketch, at fewer
# tokens as well, they give there (128 heads of 1024 tokens and 64 of 3001 are beyond, 128 of 1023 are not).
@pytest.mark.parametrize("heads,n", [(128, 1023), (128, 1024), (64, 3001)])
@pytest.mark.parametrize("kind", ["tiny rows", "tiny sketch", "infinite", "largest"])
def test_sketches_beyond_the_parts(heads, n, kind):
    """Rows of 2^-120 under a sketch of 2^75, and rows of 2^70 under one of 2^-115, to the tolerance of any rows; a sketch with an infinity makes every score
    infinite, one with the largest float leaves them finite."""
    import torch
    r = 32
    rng = np.random.default_rng(heads)
    K = rng.standard_normal((heads, n, 128)).astype(np.float32)
    G = (rng.standard_normal((128, r)) / np.sqrt(r)).astype(np.float32)
    if kind == "tiny rows":
        K, G = K * np.float32(2.0 ** -120), G * np.float32(2.0 ** 75)
    elif kind == "tiny sketch":
        K, G = K * np.float32(2.0 ** 70), G * np.float32(2.0 ** -115)
    else:
        G[17, 3] = np.inf if kind == "infinite" else np.finfo(np.float32).max
        K[..., 17] *= np.float32(2.0 ** -120)
    with B.Context(heads, 1, 4, 128, r, "fp32", n, 1, "k") as ctx:
        ctx.set_sketch(heads // 2, 0, G)
        dK = torch.from_numpy(K).cuda()
        raw, sums = torch.full((heads, n), float("nan"), device="cuda"), torch.zeros((heads,), dtype=torch.float64, device="cuda")
        ctx.scores_append(dK, dK, n, 0, n, raw, sums)
        got = raw[heads // 2].cpu().numpy()
        ctx.set_sketch(heads // 2, 0, np.ones((128, r), np.float32))        # in range again
        ctx.scores_append(dK, dK, n, 0, n, raw, sums)
        ones = raw[heads // 2].cpu().numpy()
    rows = K[heads // 2].astype(np.float64)
    if kind == "infinite":
        assert np.all(np.isposinf(got))
    else:
        want = ((rows @ G.astype(np.float64)) ** 2).sum(1)
        assert np.all(np.abs(got - want) <= PLAIN_TOL * want)
    if kind in ("infinite", "largest"):
        want = r * rows.sum(1) ** 2
        assert np.linalg.norm(ones - want) <= NORM_TOL * np.linalg.norm(want)
