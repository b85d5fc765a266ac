"""The kernel for few tokens where it takes more of them by its load (steps of a workgroup times workgroups of a compute unit): sizes around its
limits on 256 units, and the longest heads that it takes by the rule in force with the first that it does not.  Against the float64 oracle."""
import numpy as np
import pytest

from oracle import curdkv_oracle as orc
from paper_2509_15038_amd import binding as B
from tests import gpu_util as gu

pytestmark = pytest.mark.gpu

SEED = 0xC0DE0015
# some 30 roundings of 2^-24 relative to a score: sums of 128 products, their squares, sums over the columns, product and division
NORM_TOL = 1e-6


# (a step is 16 tokens; a unit holds 4, 2 or 1 workgroups at up to 32, 64 and 128 columns; 64 workgroups a head from three heads on)
@pytest.mark.parametrize("dtype,r,heads,n", [("bf16", 20, 16, 1024), ("bf16", 20, 8, 3072), ("bf16", 20, 8, 3073), ("bf16", 20, 2, 12001), ("bf16", 20, 64, 257), ("bf16", 20, 65, 257),
                                             ("bf16", 64, 16, 1024), ("bf16", 64, 16, 1025), ("bf16", 33, 32, 509), ("bf16", 128, 4, 3071), ("bf16", 128, 4, 3073),
                                             ("fp32", 20, 8, 5119), ("fp32", 20, 8, 5121), ("fp32", 32, 256, 128), ("fp32", 20, 257, 128), ("fp32", 8, 1, 40960), ("fp32", 20, 1, 40961),
                                             ("fp32", 20, 64, 1009), ("fp32", 64, 8, 4096), ("fp32", 64, 8, 4097), ("fp32", 33, 64, 500), ("fp32", 128, 8, 3072), ("fp32", 128, 8, 3073)])
@pytest.mark.parametrize("source", ["kv", "k"])
def test_scores_and_appends(dtype, r, heads, n, source):
    _check(dtype, r, heads, n, source)


def _blocks(units, dtype, r, heads, n, source, running):
    waves = (2 if source == "kv" else 1) * (2 if r <= 32 else 4 if r <= 64 else 8)
    steps = -(-n // 16)
    if steps <= 2 and (running or dtype == "bf16"):
        return 1
    places, alone = units * (16 // waves) // heads, units // heads
    return min(max(1, min(places, steps)), 64 if heads > 2 or alone < 64 else min(alone, 256))


def _taken(units, dtype, r, heads, n, source, running):
    """Whether the kernel for few tokens takes a call of more tokens than one of its steps."""
    steps, blocks = -(-n // 16), _blocks(units, dtype, r, heads, n, source, running)
    if dtype == "fp32":
        always = n * heads <= FEW_F32 and steps <= STEPS_F32 * blocks
        most, load = (units // 2 if running or source != "kv" else HEADS_F32), LOAD_F32
    else:
        always = n * heads <= FEW_BF16 // ((1 if r <= 32 else 2 if r <= 64 else 4) if heads > units // 4 else 1) and steps <= STEPS_BF16 * blocks
        most, load = LIMITS_BF16[0 if r <= 32 else 1 if r <= 64 else 2]
    return always or (heads <= most and -(-steps // blocks) * -(-blocks * heads // units) <= load)


LIMITS_BF16 = [(gu.limit("scores_kernels.hip", "kFewHeadsBf16" + w), gu.limit("scores_kernels.hip", "kFewLoadBf16" + w)) for w in ("", "Mid", "Wide")]
HEADS_F32, LOAD_F32 = gu.limit("scores_kernels.hip", "kFewHeadsF32"), gu.limit("scores_kernels.hip", "kFewLoadF32")
FEW_F32, STEPS_F32 = gu.limit("scores_kernels.hip", "kFewF32Tokens"), gu.limit("scores_kernels.hip", "kFewF32Steps")
FEW_BF16, STEPS_BF16 = gu.limit("scores_kernels.hip", "kFewBf16Tokens"), gu.limit("scores_kernels.hip", "kFewBf16Steps")


# heads: few, and the most that the rule takes (and one more, which it takes only by the tokens in all): of both sources, or of one
@pytest.mark.parametrize("dtype,r,heads", [("bf16", 20, 1), ("bf16", 20, 8), ("bf16", 32, 64), ("bf16", 20, 65), ("bf16", 33, 8), ("bf16", 64, 32), ("bf16", 64, 33), ("bf16", 65, 8),
                                           ("bf16", 128, 32), ("fp32", 20, 1), ("fp32", 32, 8), ("fp32", 20, 100), ("fp32", 20, 128), ("fp32", 20, 129), ("fp32", 8, 200), ("fp32", 20, 256), ("fp32", 20, 257)])
@pytest.mark.parametrize("source", ["kv", "k"])
def test_both_sides_of_the_rule(dtype, r, heads, source):
    import torch
    units = torch.cuda.get_device_properties(0).multi_processor_count
    for running in (False, True):
        last = max(n for n in range(40, 60000 // heads + 300) if _taken(units, dtype, r, heads, n, source, running) or n == 40)
        if last < 300 and running and dtype == "bf16":
            continue                                                     # (one workgroup a head with the sum in it: test_gpu_bf16_few.py)
        for n in (last, last + 1):
            few = _taken(units, dtype, r, heads, n, source, running)
            kernel = _check(dtype, r, heads, n, source)[running][0]
            assert (kernel == "scores_few_kernel") == few, (dtype, r, heads, n, source, running, kernel)


def _check(dtype, r, heads, n, source):
    """Scores and appends, once and again behind themselves; returns the kernels that scored (alone, with a running sum)."""
    import torch
    dt = torch.bfloat16 if dtype == "bf16" else torch.float32
    g = torch.Generator(device="cuda")
    g.manual_seed(n * 512 + r)
    K = (torch.randn((heads, n, 128), generator=g, device="cuda") * torch.exp(torch.randn((heads, 1, 128), generator=g, device="cuda"))).to(dt)
    V = (torch.randn((heads, n, 128), generator=g, device="cuda") * torch.exp(torch.randn((heads, n, 1), generator=g, device="cuda"))).to(dt)
    with B.Context(heads, 1, 4, 128, r, dtype, 2 * n, SEED, source) as ctx:
        out = gu.Guarded((heads, n), torch.float32, float("nan"))
        ctx.scores(K, V, n, out.t)
        raw, sums = gu.Guarded((heads, 2 * n), torch.float32, float("nan")), torch.full((heads,), 7.0, dtype=torch.float64, device="cuda")
        ctx.scores_append(K, V, n, 0, 2 * n, raw.t, sums)
        once = sums.cpu().numpy().copy()
        kernels = [gu.launches(lambda: ctx.scores(K, V, n, out.t))[0], gu.launches(lambda: ctx.scores_append(K, V, n, 0, 2 * n, raw.t, sums))[0]]
        ctx.scores_append(K, V, n, n, 2 * n, raw.t, sums)                # the same tokens again behind the first: the sum doubles
        torch.cuda.synchronize()
        out.check("scores"), raw.check("raw")
        out, raw, sums = out.t.cpu().numpy(), raw.t.cpu().numpy().astype(np.float64), sums.cpu().numpy()
    assert np.array_equal(raw[:, :n], raw[:, n:]) and np.allclose(once, raw[:, :n].sum(1), rtol=1e-6) and np.allclose(sums, 2 * once, rtol=1e-12)
    for i in (0, heads // 2, heads - 1):
        G = orc.sketch(SEED, i, 0, 1, 128, r, dtype)
        want = orc.scores(K[i].double().cpu().numpy(), V[i].double().cpu().numpy(), G, source)
        for x in (out[i], raw[i, :n] / once[i]):
            assert np.linalg.norm(x - want) <= NORM_TOL * np.linalg.norm(want), (dtype, r, heads, n, source, i)
    return kernels
