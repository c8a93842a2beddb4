"""GPU parity of folded properties: the enumeration on a property's reduced
network (constant neurons folded into the biases, ibmc_set_variant "fold")
must return the oracle's counts, ties and records exactly.  The shapes reach
every compiled first-layer width (32 to 256 live units), layer-2 tile counts
with and without a remainder, both requantiser forms, products that need the
saturating sum or a halved scale, logit differences beyond one byte, segments
shorter than a tile, and one to three perturbed pixels."""
import numpy as np
import pytest

from paper_1907_12933_amd import inputs as I

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    from paper_1907_12933_amd import ibmc
    return ibmc.Context(0)


def live_net(g, dims, shift, wmax, spread):
    """A net whose first-layer potentials at a mid-grey image lie within
    `spread` windows of the requantiser's, so that many units are live."""
    net = I.random_qnet(g, dims, shift=shift, wmax=wmax, bmax=300)
    win = 128 << net.shift[0]
    c = g.uniform(0.5 - spread, 0.5 + spread, size=dims[1]) * win
    net.b[0] = (c - net.W[0].astype(np.int64) @ np.full(dims[0], 128)).astype(np.int32)
    return net


# (dims, shifts, wmax, spread, deltas, k_min, k_max)
CASES = [
    ([18, 16, 5], [7], 64, 0.5, [-16, 16], 0, 3),             # at most 32 units, one hidden layer
    ([9, 30, 2], [3], 20, 0.5, [5], 1, 2),                    # one delta; segments of a few positions
    ([20, 70, 10], [6], 64, 0.4, [-60, -5, 5, 60], 1, 2),     # 64 / 128 wide, saturating sum
    ([24, 250, 16], [8], 127, 0.5, [-40, 9, 40], 1, 2),       # 256 wide, 16 classes, two-byte differences
    ([16, 40, 30, 6], [5, 4], 40, 0.6, [-255, 255], 1, 3),    # general requantiser, halved scale
    ([30, 64, 64, 10], [7, 7], 64, 0.5, [-60, 30], 1, 2),     # saturating epilogue
    ([14, 100, 90, 7], [7, 7], 127, 0.5, [-90, 3, 90], 1, 2),  # 128 wide, remainder tiles
    ([12, 256, 200, 10], [6, 8], 64, 0.5, [-32, 32], 1, 2),   # 256 wide, second shift 8
    ([22, 33, 250, 4], [0, 7], 3, 0.5, [-200, 200], 1, 2),    # shift 0, 16 layer-2 tiles
    ([25, 64, 17, 3], [8, 2], 127, 0.5, list(range(-16, 17)), 1, 2),  # 33 deltas: five groups of segments
]


@pytest.mark.parametrize("seed", range(len(CASES)))
def test_folded_check_equals_the_oracle(ctx, orc, seed):
    from paper_1907_12933_amd import ibmc
    dims, shift, wmax, spread, deltas, k0, k1 = CASES[seed]
    g = I.rng(900 + seed)
    net = live_net(g, dims, shift, wmax, spread)
    D = np.array(deltas, np.int16)
    m = ibmc.Mlp(ctx, net)
    ibmc.ibmc_set_variant(ctx, m, "fold")
    assert ibmc.ibmc_chosen_variant(ctx, m) == "fold"
    # a mid-grey image and one with saturated pixels, as one batch, so that a
    # workgroup changes property
    xs = [g.integers(96, 160, size=dims[0]).astype(np.uint8), g.integers(0, 255, size=dims[0], endpoint=True).astype(np.uint8)]
    xs[1][:3] = [0, 255, 128]
    sums, recs, _, _ = ibmc.ibmc_check_batch(ctx, [(m, x, D, k0, k1) for x in xs], cex_capacity=1 << 21)
    for i, x in enumerate(xs):
        r = orc.q8_check(net, x, D, k0, k1, cap=1 << 21)
        c = recs[recs["prop"] == i]
        assert sums[i]["clean_label"] == r["clean_label"]
        assert list(sums[i]["cex"]) == [int(v) for v in r["cex"]]
        assert list(sums[i]["ties"]) == [int(v) for v in r["ties"]]
        assert np.array_equal(c["k"], r["cex_k"]) and np.array_equal(c["rank"], r["cex_rank"])
        assert np.array_equal(c["new_label"], r["cex_label"])


def test_some_case_has_counterexamples_and_ties(orc):
    """The cases above are not all safe (checked on the oracle alone)."""
    cex = 0
    for seed, (dims, shift, wmax, spread, deltas, k0, _) in enumerate(CASES):
        g = I.rng(900 + seed)
        net = live_net(g, dims, shift, wmax, spread)
        x = g.integers(96, 160, size=dims[0]).astype(np.uint8)
        cex += orc.q8_check(net, x, np.array(deltas, np.int16), 1, 2)["cex_total"] > 0
    assert cex >= 3


def test_mixed_batch_and_truncation(ctx, orc):
    """Folded and unfolded networks in one call (several instances beside each
    other), host and device images, a capacity below the number of records,
    and the same call again."""
    import torch
    from paper_1907_12933_amd import ibmc
    g = I.rng(950)
    specs = [([18, 16, 5], [7]), ([30, 64, 64, 10], [7, 7]), ([14, 100, 90, 7], [7, 7]), ([20, 70, 10], [6])]
    nets = [live_net(g, d, s, 64, 0.5) for d, s in specs]
    D = np.array([-60, -20, 20, 60], np.int16)
    ms = [ibmc.Mlp(ctx, n) for n in nets]
    for i, m in enumerate(ms):
        if i != 2:
            ibmc.ibmc_set_variant(ctx, m, "fold")   # the third keeps its own kernel
    xs = [g.integers(96, 160, size=n.dims[0]).astype(np.uint8) for n in nets for _ in range(2)]
    props = [(ms[i // 2], x, D, 1, 2) for i, x in enumerate(xs)]
    refs = [orc.q8_check(nets[i // 2], x, D, 1, 2, cap=1 << 20) for i, x in enumerate(xs)]
    total = sum(r["cex_total"] for r in refs)
    assert total > 100
    for on_device, cap in ((False, 1 << 20), (True, 1 << 20), (False, total // 2)):
        P = [(m, torch.from_numpy(x).cuda() if on_device else x, *rest) for m, x, *rest in props]
        for _ in range(2):
            sums, recs, _, rc = ibmc.ibmc_check_batch(ctx, P, cex_capacity=cap, on_device=on_device)
            assert rc == (ibmc.IBMC_W_TRUNCATED if cap < total else ibmc.IBMC_OK) and len(recs) == min(cap, total)
            for i, r in enumerate(refs):
                assert list(sums[i]["cex"]) == [int(v) for v in r["cex"]]
                c = recs[recs["prop"] == i]
                if cap >= total:
                    assert np.array_equal(c["rank"], r["cex_rank"]) and np.array_equal(c["new_label"], r["cex_label"])
                else:
                    assert set(zip(c["k"], c["rank"])) <= set(zip(r["cex_k"], r["cex_rank"]))
