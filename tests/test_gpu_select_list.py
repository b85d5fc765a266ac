"""The selection's list of candidates in the cut bin: its sizes around 32 keys (compared with
each other) and beyond (resolved digit by digit), with ties across the cut, exact against the oracle; and heads whose partial sums, lengths and offsets leave waves partly idle in the normalisation."""
import numpy as np
import pytest

from oracle import curdkv_oracle as orc
from paper_2509_15038_amd import binding as B

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [3000, 9001, 33000])       # 4, 16 and 36 keys per thread
@pytest.mark.parametrize("inside", [1, 2, 31, 32, 33, 64, 200])
def test_cut_bin_of_every_size(n, inside):
    """`inside` candidates share the bin [1, 1 + 1/32) with the threshold, half of them drawn from eight values."""
    import torch
    rng = np.random.Generator(np.random.PCG64([n, inside]))
    above, heads = 100, 6
    scores = rng.uniform(0.0, 0.5, (heads, n)).astype(np.float32)
    budgets = np.zeros((heads,), np.int32)
    for h in range(heads):
        place = rng.permutation(np.arange(4, n))
        scores[h, place[:above]] = rng.uniform(1.5, 1.9, above)
        fine = rng.uniform(1.0, 1.03, inside)
        coarse = 1.0 + rng.integers(0, 8, inside) / 512.0
        scores[h, place[above:above + inside]] = np.where(rng.random(inside) < 0.5, fine, coarse)
        rank = (1, inside, (inside + 1) // 2, rng.integers(1, inside + 1), 1, inside)[h]
        budgets[h] = 4 + above + rank
    offsets = np.concatenate([[0], np.cumsum(budgets, dtype=np.int64)])
    with B.Context(1, heads, 4, 128, 20, "bf16", n, 1) as ctx:
        out = torch.full((int(offsets[-1]),), -1, dtype=torch.int32, device="cuda")
        ctx.select(torch.from_numpy(scores).cuda(), n, budgets, 4, offsets, out)
        out = out.cpu().numpy()
    for h in range(heads):
        want = orc.select(scores[h], int(budgets[h]), 4)
        assert np.array_equal(out[offsets[h]:offsets[h + 1]], want), (n, inside, h)


# the sizes around which threads are dealt differently to the keys and to the parts of the others that they are compared
# with, and where the digits take over
@pytest.mark.parametrize("n", [3000, 33000])
@pytest.mark.parametrize("inside", [47, 48, 49, 63, 65, 127, 128, 129])
def test_cut_bin_compared_in_parts(n, inside):
    test_cut_bin_of_every_size(n, inside)


@pytest.mark.parametrize("n", [1, 2, 63, 65, 255, 257, 1025, 2049, 4099])
@pytest.mark.parametrize("heads", [1, 5])
def test_normalised_scores_add_up(n, heads):
    """bf16 scores sum to one per head from both normalisations, and agree (one rounding of the sum apart)."""
    import torch
    g = torch.Generator(device="cuda")
    g.manual_seed(n * 8 + heads)
    K = torch.randn((heads, n, 128), generator=g, device="cuda").to(torch.bfloat16)
    V = torch.randn((heads, n, 128), generator=g, device="cuda").to(torch.bfloat16)
    with B.Context(1, heads, 4, 128, 64, "bf16", n, 3) as ctx:
        one = torch.full((heads, n), float("nan"), device="cuda")
        ctx.scores(K, V, n, one)
        raw, two = torch.empty_like(one), torch.full_like(one, float("nan"))
        sums = torch.zeros((heads,), dtype=torch.float64, device="cuda")
        ctx.scores_append(K, V, n, 0, n, raw, sums)
        ctx.normalise(raw, sums, n, n, two)
        one, two = one.double().cpu(), two.double().cpu()
    # 4099 terms and a division, each rounded to 2^-24 of its size
    assert torch.allclose(one.sum(1), torch.ones(heads, dtype=torch.float64), rtol=0, atol=4e-7)
    assert torch.allclose(one, two, rtol=4e-7, atol=0)
