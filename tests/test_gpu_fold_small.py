"""Calls of many small properties, whose networks are folded or not by their
mean number of points: on both sides of the line, and a network above it beside
one below it in one call, the results are those of the networks' own kernels
and, for some properties, the oracle's."""
import numpy as np
import pytest

from paper_1907_12933_amd import inputs as I

pytestmark = pytest.mark.gpu

# (dims, shifts, properties, deltas): 35-32-16-5 is folded from 400 points a
# property on, 20-24-5 (no lane kernel by itself) from 200
CASES = {
    "three layers below": [([35, 32, 16, 5], [7, 7], 230, 11)],
    "three layers above": [([35, 32, 16, 5], [7, 7], 230, 12)],
    "two layers below": [([20, 24, 5], [7], 170, 9)],
    "two layers above": [([20, 24, 5], [7], 170, 10)],
    "both": [([35, 32, 16, 5], [7, 7], 100, 11), ([20, 24, 5], [7], 170, 10)],
}


@pytest.mark.parametrize("case", sorted(CASES))
def test_mean_points(orc, case):
    from paper_1907_12933_amd import ibmc
    ctx = ibmc.Context(0)
    g = I.rng(len(case))
    nets, ms, P = [], [], []
    for dims, shift, count, deltas in CASES[case]:
        nets.append(I.random_qnet(g, dims, shift=shift))
        ms.append(ibmc.Mlp(ctx, nets[-1]))
        D = (np.arange(deltas) * 9 - 50).astype(np.int16)
        X = g.integers(0, 255, size=(count, dims[0]), endpoint=True).astype(np.uint8)
        P += [(ms[-1], x, D, 1, 1) for x in X]

    def run():
        sums, recs, _, rc = ibmc.ibmc_check_batch(ctx, P, cex_capacity=1 << 18)
        assert rc == ibmc.IBMC_OK
        return [(s["clean_label"], s["cex"], s["ties"]) for s in sums], recs

    got = run()
    for m in ms:
        ibmc.ibmc_set_variant(ctx, m, ibmc.ibmc_chosen_variant(ctx, m))
    plain = run()
    assert got[0] == plain[0] and np.array_equal(got[1], plain[1]) and len(got[1]) > 0
    for i in (0, len(P) // 2, len(P) - 1):
        r = orc.q8_check(nets[ms.index(P[i][0])], P[i][1], P[i][2], 1, 1)
        assert got[0][i][0] == r["clean_label"] and list(got[0][i][1]) == list(r["cex"]) and list(got[0][i][2]) == list(r["ties"])
        c = got[1][got[1]["prop"] == i]
        assert np.array_equal(c["rank"], r["cex_rank"]) and np.array_equal(c["new_label"], r["cex_label"])
