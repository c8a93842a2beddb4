"""GPU check of the record lists around the edges of the single-workgroup
sort: 1 to 16,380 counterexamples (one below, at and above the powers of two
where its padding changes, and above its longest list, where the radix sort
takes over), in host and in device memory, must be the oracle's list, in its
order.  All-integer, so equality is exact."""
import numpy as np
import pytest

from paper_1907_12933_amd import inputs as I

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    from paper_1907_12933_amd import ibmc
    return ibmc.Context(0)


def sum_net(n, hidden, limit):
    """Label 1 as soon as the pixels' sum exceeds the mid-grey image's by more
    than `limit`, else label 0 (a sum of exactly `limit` is a tie)."""
    net = I.random_qnet(I.rng(7), [n, hidden, 5], shift=0, wmax=1, bmax=1)
    net.W[0][:] = 1
    net.b[0][:] = -128 * n
    net.W[1][:] = 0
    net.W[1][1, 0] = 1
    net.b[1][:] = [limit, 0, -1, -1, -1]
    return net


# (pixels, hidden units, deltas, k): every point with a delta above 4 is a counterexample
CASES = [
    (1, 16, [5], 1), (63, 16, [9], 1), (64, 32, [9], 1), (65, 16, [9], 1),
    (64, 16, list(range(5, 37)), 1), (89, 32, list(range(5, 28)), 1),     # 2,048 and 2,047
    (64, 16, list(range(5, 69)), 1), (241, 16, list(range(5, 22)), 1),    # 4,096 and 4,097
    (64, 32, [5, 6], 2), (91, 16, [6, 7], 2), (65, 16, [5, 6], 2),        # 8,064, 16,380 and 8,320
]


@pytest.mark.parametrize("n,hidden,deltas,k", CASES)
def test_short_lists(ctx, orc, n, hidden, deltas, k):
    import torch
    from paper_1907_12933_amd import ibmc
    net = sum_net(n, hidden, 4)
    m = ibmc.Mlp(ctx, net)
    x = np.full(n, 128, np.uint8)
    D = np.array([-3, 4] + deltas if k == 1 and len(deltas) < 60 else deltas, np.int16)
    r = orc.q8_check(net, x, D, k, k, cap=1 << 20)
    assert r["cex_total"] >= len(deltas) * n
    for variant in (None, "fold"):
        ibmc.ibmc_set_variant(ctx, m, variant)
        for cap in (1 << 16, max(1, r["cex_total"] - 1)):
            sums, recs, _, _ = ibmc.ibmc_check_batch(ctx, [(m, x, D, k, k)], cex_capacity=cap)
            assert list(sums[0]["cex"]) == [int(v) for v in r["cex"]]
            assert list(sums[0]["ties"]) == [int(v) for v in r["ties"]]
            assert len(recs) == min(cap, r["cex_total"])
            if cap >= r["cex_total"]:
                assert np.array_equal(recs["rank"], r["cex_rank"]) and np.array_equal(recs["new_label"], r["cex_label"])
            else:
                assert set(recs["rank"]) <= set(r["cex_rank"]) and np.all(np.diff(recs["rank"]) > 0)
        buf = torch.empty((1 << 16) * 24, dtype=torch.uint8, device="cuda")
        sums, _, _, _ = ibmc.ibmc_check_batch(ctx, [(m, x, D, k, k)], cex_capacity=1 << 16, cex_buf=buf,
                                              records_on_device=True)
        got = buf.cpu().numpy().view(ibmc.CEX_DTYPE)[:r["cex_total"]]
        assert np.array_equal(got["rank"], r["cex_rank"]) and np.array_equal(got["new_label"], r["cex_label"])
        assert np.all(got["prop"] == 0) and np.all(got["k"] == k)
