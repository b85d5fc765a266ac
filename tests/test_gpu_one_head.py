"""One or two heads: scored by more than 64 workgroups each, whose partial sums are then several to a lane.  Scores and sums
against 64 bits, indices against the oracle's selection on the scores as stored."""
import numpy as np
import pytest

from oracle import curdkv_oracle as orc
from paper_2509_15038_amd import binding as B
from paper_2509_15038_amd import workloads as wl
from tests import gpu_util as gu

pytestmark = pytest.mark.gpu


# A score errs by 2e-7 at root mean square with 20 columns and 9e-8 with more (roundings of 128 products' sums, squared, twice): seven
# times that over the 260000 scores compared, and twice that again.  A sum of scores: chains of up to 64 fp32 additions, at random.
SCORE_TOL, SUM_TOL = {20: 48 * 2.0 ** -24, 64: 24 * 2.0 ** -24, 128: 24 * 2.0 ** -24}, 1e-6


# A wave has two 32-token tiles at least: 256 workgroups from 65536 tokens on.  (8192: tokens that the few-token kernel takes whatever its load, 24576 + 1: the split
# selection's line; 2 heads of 3000 and 3 of 3000: the few-token kernel's workgroups are as many as units, or 64 a head)
@pytest.mark.parametrize("heads,n", [(2, 3000), (3, 3000), (1, 4096), (1, 8192), (1, 8193), (1, 16640), (1, 24577), (2, 24577), (1, 40001), (2, 49153), (1, 65537), (2, 100003), (1, 131072), (1, 131073)])
@pytest.mark.parametrize("r,dtype", [(20, "bf16"), (128, "bf16"), (20, "fp32"), (64, "fp32")])
def test_scores_sums_and_selection(heads, n, r, dtype):
    import torch
    g = torch.Generator(device="cuda")
    g.manual_seed(n + r)
    dt = torch.bfloat16 if dtype == "bf16" else torch.float32
    K = torch.randn((1, heads, n, 128), generator=g, device="cuda").to(dt)
    V = (torch.randn((1, heads, n, 128), generator=g, device="cuda") * torch.randn((1, heads, n, 1), generator=g, device="cuda").exp()).to(dt)
    with B.Context(1, heads, 4, 128, r, dtype, n, 11) as ctx:
        G = torch.stack([torch.from_numpy(orc.sketch(11, 0, h, heads, 128, r, dtype)) for h in range(heads)]).cuda().double()
        want = torch.stack([(K[0, h].double() @ G[h]).square_().sum(1) * (V[0, h].double() @ G[h]).square_().sum(1) for h in range(heads)])
        raw = gu.Guarded((heads, n), torch.float32, float("nan"))
        sums = torch.zeros((heads,), dtype=torch.float64, device="cuda")
        ctx.scores_append(K, V, n, 0, n, raw.t, sums)
        assert torch.allclose(raw.t.double(), want, rtol=SCORE_TOL[r], atol=0)
        assert torch.allclose(sums, raw.t.double().sum(1), rtol=SUM_TOL, atol=0)
        for k, s in ((n // 10, 4), (n // 2, 0)):
            budgets = np.full((heads,), k, dtype=np.int32)
            off = wl.offsets_for(budgets)
            for one_call in (True, False):
                sc, idx, Ko, Vo, _ = gu.run_path(ctx, K, V, n, budgets, s, dtype, one_call=one_call)
                assert torch.allclose(sc.double(), want / want.sum(1, keepdim=True), rtol=SCORE_TOL[r] + 2 * SUM_TOL, atol=0)
                where = idx.long()
                for h in range(heads):
                    mine = slice(int(off[h]), int(off[h + 1]))
                    assert np.array_equal(where[mine].cpu().numpy(), orc.select(sc[h].cpu().numpy().astype(np.float64), k, s))
                    assert torch.equal(Ko[mine], K[0, h, where[mine]]) and torch.equal(Vo[mine], V[0, h, where[mine]])
        raw.check()
