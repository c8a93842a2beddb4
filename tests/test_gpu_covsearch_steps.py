"""Test generation at the edges of the search kernels: a cap on the tests just
below, at and above the number of greedy steps queued at a time (16), layers
of 1 to 64 units (the packed weight words' remainders), one and four weight
layers, against the greedy selection over the oracle's per-pair coverage."""
import numpy as np
import pytest

from paper_1907_12933_amd import inputs as I
from test_gpu_covsearch import oracle_greedy

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    from paper_1907_12933_amd import ibmc
    return ibmc.Context(0)


@pytest.mark.parametrize("dims,shift,crit,caps", [
    ([20, 33, 31, 5], [4, 3], "SS", (1, 2, 15, 16, 17, 33)),
    ([17, 64, 60, 3], [4, 4], "DV", (1, 16, 64)),
    ([16, 9, 17, 6, 2], [3, 3, 2], "SV", (2, 16, 40)),
    ([25, 1, 4], [3], "DS", (1, 3)),
])
def test_search_steps(ctx, orc, dims, shift, crit, caps):
    from paper_1907_12933_amd import ibmc
    g = I.rng(sum(dims))
    net = I.random_qnet(g, dims, shift=shift, wmax=40, bmax=300)
    m = ibmc.Mlp(ctx, net)
    x = g.integers(0, 255, size=dims[0], endpoint=True).astype(np.uint8)
    D = np.array([-120, -60, -20, 20, 60, 120], np.int16)
    for cap in caps:
        seq, covered, union = oracle_greedy(orc, net, x, D, 1, crit, cap)
        tests, gains, cov = ibmc.ibmc_coverage_search(ctx, m, x, D, 1, crit, max_tests=cap)
        assert [(int(t["rank"]), int(gn), int(t["new_label"])) for t, gn in zip(tests, gains)] == seq
        assert np.array_equal(cov["bits"], covered)
        assert cov["covered_pairs"] == sum(s[1] for s in seq)
