"""The kernel for few tokens where it takes more of them by its load (steps of a workgroup times workgroups of a compute unit), on both sides
of each limit, and the plain fp32 kernel beyond it.  Against the float64 oracle."""
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
