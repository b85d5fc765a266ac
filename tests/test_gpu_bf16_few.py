"""bf16 calls of few tokens in all: workgroups of 16 tokens whose waves share the products.  Scores and
running sums against the float64 oracle at the edges of the 16-token steps, with one step and several
per workgroup, and around the lines where the kernel of longer calls takes over."""
import numpy as np
import pytest

from oracle import curdkv_oracle as orc
from paper_2509_15038_amd import binding as B

pytestmark = pytest.mark.gpu

SEED = 0xC0DE0011
# products of bf16 numbers are exact; a projected coordinate is rounded once per 32 of them, then squared,
# summed over r, multiplied and normalised: some 200 roundings of 2^-24 at random, and the sums' own
NORM_TOL = 1e-6


# one token; edges of a step; two steps in one workgroup and three in three; 64 workgroups of 1 and 4 steps and one step more; many heads, around
# the tokens up to which each width is taken (beyond them a call may be taken by its load: test_gpu_few_load.py asks which kernel runs)
@pytest.mark.parametrize("n,heads", [(1, 1), (16, 1), (17, 3), (32, 2), (33, 2), (1025, 1), (4096, 1), (4097, 1), (1, 256),
                                     (8, 256), (9, 256), (32, 256), (33, 256), (1024, 8), (1025, 8)])
@pytest.mark.parametrize("r,source", [(20, "kv"), (33, "v"), (64, "kv"), (128, "k"), (128, "kv")])
def test_scores_and_sums(n, heads, r, source):
    import torch
    g = torch.Generator(device="cuda")
    g.manual_seed(n * 512 + heads)
    K = torch.randn((heads, n, 128), generator=g, device="cuda").to(torch.bfloat16)
    V = torch.randn((heads, n, 128), generator=g, device="cuda").to(torch.bfloat16)
    with B.Context(heads, 1, 4, 128, r, "bf16", n + 7, SEED, source) as ctx:
        got = torch.full((heads, n), float("nan"), device="cuda")
        ctx.scores(K, V, n, got)
        # behind five tokens scored before, in rows of n + 7 places: only the new ones are written
        raw = torch.full((heads, n + 7), -1.0, device="cuda")
        sums = torch.full((heads,), 3.0, dtype=torch.float64, device="cuda")
        ctx.scores_append(K, V, n, 5, n + 7, raw, sums)
        got, raw, sums = got.cpu().numpy(), raw.cpu().numpy(), sums.cpu().numpy()
    assert np.all(raw[:, :5] == -1.0) and np.all(raw[:, n + 5:] == -1.0)
    assert np.allclose(sums - 3.0, raw[:, 5:n + 5].astype(np.float64).sum(1), rtol=1e-6)
    for i in range(heads) if heads < 8 else (0, heads // 2, heads - 1):
        G = orc.sketch(SEED, i, 0, 1, 128, r, "bf16")
        want = orc.scores(K[i].double().cpu().numpy(), V[i].double().cpu().numpy(), G, source)
        assert np.linalg.norm(got[i] - want) <= NORM_TOL * np.linalg.norm(want), (n, heads, r, source, i)
        new = raw[i, 5:n + 5].astype(np.float64)
        assert np.linalg.norm(new / new.sum() - want) <= NORM_TOL * np.linalg.norm(want)


def _launches(call):
    """Kernels that `call` launches, as nodes of a captured graph."""
    import ctypes
    import torch
    graph = torch.cuda.CUDAGraph(keep_graph=True)
    with torch.cuda.graph(graph):
        call()
    path = next(line.split()[-1] for line in open("/proc/self/maps") if "libamdhip64" in line)
    count = ctypes.c_size_t()
    assert ctypes.CDLL(path).hipGraphGetNodes(ctypes.c_void_p(graph.raw_cuda_graph()), None, ctypes.byref(count)) == 0
    return count.value


# both sides of the tokens from which the kernel of longer calls takes appends (8, 16 or 32 by width), of the step from one
# workgroup per head to several in it (256), and of the line where 128 columns are split all the same (192)
@pytest.mark.parametrize("r", [20, 33, 64, 128])
@pytest.mark.parametrize("n", [1, 8, 9, 16, 17, 32, 33, 64, 128, 192, 193, 256, 257])
@pytest.mark.parametrize("heads", [1, 8])
def test_short_appends(n, heads, r):
    """Raw scores and running sums, and a single launch wherever one workgroup per head can add its sum by itself."""
    import torch
    g = torch.Generator(device="cuda")
    g.manual_seed(n * 512 + r)
    K = torch.randn((heads, n, 128), generator=g, device="cuda").to(torch.bfloat16)
    V = torch.randn((heads, n, 128), generator=g, device="cuda").to(torch.bfloat16)
    with B.Context(heads, 1, 4, 128, r, "bf16", n + 5, SEED) as ctx:
        raw = torch.full((heads, n + 5), -1.0, device="cuda")
        sums = torch.full((heads,), 3.0, dtype=torch.float64, device="cuda")
        ctx.scores_append(K, V, n, 5, n + 5, raw, sums)
        torch.cuda.synchronize()
        scores, total = raw.cpu().numpy(), sums.cpu().numpy()
        launches = _launches(lambda: ctx.scores_append(K, V, n, 5, n + 5, raw, sums))
    assert launches == (1 if n <= (256 if r <= 64 else 192) else 2)
    assert np.all(scores[:, :5] == -1.0)
    assert np.allclose(total - 3.0, scores[:, 5:].astype(np.float64).sum(1), rtol=1e-6)
    for i in (0, heads - 1):
        G = orc.sketch(SEED, i, 0, 1, 128, r, "bf16")
        want = orc.scores(K[i].double().cpu().numpy(), V[i].double().cpu().numpy(), G)
        new = scores[i, 5:].astype(np.float64)
        assert np.linalg.norm(new / new.sum() - want) <= NORM_TOL * np.linalg.norm(want)


# numbers of heads that do not divide the chip's places; two steps; 64 columns in many heads on both sides of 4096 tokens
@pytest.mark.parametrize("heads,n", [(12, 576), (17, 300), (4, 25), (224, 19), (100, 40), (100, 41), (129, 31)])
@pytest.mark.parametrize("r", [20, 64, 128])
@pytest.mark.parametrize("dtype", ["bf16", "fp32"])
def test_numbers_of_heads(heads, n, r, dtype):
    import torch
    g = torch.Generator(device="cuda")
    g.manual_seed(n * 512 + r)
    tdt = torch.bfloat16 if dtype == "bf16" else torch.float32
    K = torch.randn((heads, n, 128), generator=g, device="cuda").to(tdt)
    V = torch.randn((heads, n, 128), generator=g, device="cuda").to(tdt)
    with B.Context(heads, 1, 4, 128, r, dtype, n, SEED) as ctx:
        got, raw = torch.full((heads, n), float("nan"), device="cuda"), torch.full((heads, n), float("nan"), device="cuda")
        sums = torch.zeros((heads,), dtype=torch.float64, device="cuda")
        ctx.scores(K, V, n, got)
        ctx.scores_append(K, V, n, 0, n, raw, sums)
        got, raw, sums = got.cpu().numpy(), raw.cpu().numpy().astype(np.float64), sums.cpu().numpy()
    assert np.allclose(sums, raw.sum(1), rtol=1e-6)
    for i in (0, heads // 2, heads - 1):
        G = orc.sketch(SEED, i, 0, 1, 128, r, dtype)
        want = orc.scores(K[i].double().cpu().numpy(), V[i].double().cpu().numpy(), G)
        for x in (got[i], raw[i] / raw[i].sum()):
            assert np.linalg.norm(x - want) <= NORM_TOL * np.linalg.norm(want)
