"""Folded levels cut into jobs (a level beyond 2^31 points; here the limit is
lowered for the context, so that small levels are cut at every last-prefix
pixel): one level of more than 64 jobs and calls of 64 to more than 4,096
jobs return the counts, ties and records of the unfolded kernels, whose parity
with the oracle the other tests establish, and the oracle's for one image."""
import numpy as np
import pytest

from paper_1907_12933_amd import inputs as I

pytestmark = pytest.mark.gpu

# (dims, shifts, deltas, k_max, images): jobs per image, a level of k = 1
# being one job, of k = 2 pixels - 1, of k = 3 pixels - 2
CASES = [
    ([40, 64, 5], [7], [-16, 16], 3, 1),                # 1 + 39 + 38 = 78
    ([72, 24, 20, 6], [7, 7], [-40, 40], 2, 2),         # 72 each
    ([72, 64, 5], [6], [-16, 16], 2, 56),               # 4,032
    ([72, 64, 5], [6], [-16, 16], 2, 57),               # 4,104
    ([72, 24, 20, 6], [7, 6], [-40, 40], 2, 70),        # 5,040
]


@pytest.mark.parametrize("case", range(len(CASES)))
def test_cut_levels(orc, monkeypatch, case):
    from paper_1907_12933_amd import ibmc
    dims, shift, deltas, k, count = CASES[case]
    monkeypatch.setenv("IBMC_FOLD_JOB_POINTS", "1")
    ctx = ibmc.Context(0)
    g = I.rng(70 + case)
    net = I.random_qnet(g, dims, shift=shift)
    m = ibmc.Mlp(ctx, net)
    D = np.array(deltas, np.int16)
    X = g.integers(0, 255, size=(count, dims[0]), endpoint=True).astype(np.uint8)
    P = [(m, x, D, 1, k) for x in X]
    plain = ibmc.ibmc_chosen_variant(ctx, m)
    got = {}
    for variant in ("fold", plain):
        ibmc.ibmc_set_variant(ctx, m, variant)
        sums, recs, _, rc = ibmc.ibmc_check_batch(ctx, P, cex_capacity=1 << 21)
        assert rc == ibmc.IBMC_OK
        got[variant] = ([(s["clean_label"], s["cex"], s["ties"]) for s in sums], recs)
    assert got["fold"][0] == got[plain][0] and np.array_equal(got["fold"][1], got[plain][1])
    r = orc.q8_check(net, X[-1], D, 1, k, cap=1 << 21)
    label, cex, ties = got["fold"][0][-1]
    assert label == r["clean_label"] and list(cex) == list(r["cex"]) and list(ties) == list(r["ties"])
    c = got["fold"][1][got["fold"][1]["prop"] == count - 1]
    assert np.array_equal(c["rank"], r["cex_rank"]) and np.array_equal(c["new_label"], r["cex_label"])
