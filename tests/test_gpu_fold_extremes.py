"""Folded properties whose output layer holds both ends of int8: a class weight
of 127 against a label weight of -128 on a live unit is a logit difference of
255, which no two signed bytes add up to; the opposite pair (-255) and a
difference of 254 do fit.  Counts, ties and records must equal the oracle's
exhaustive check (Sec. III-C) in each case, for one and two hidden layers."""
import numpy as np
import pytest

from paper_1907_12933_amd import inputs as I

pytestmark = pytest.mark.gpu

# (weight of the other class, weight of the label)
PAIRS = [(127, -128), (126, -128), (-128, 127)]
DIMS = [([16, 40, 5], [6]), ([14, 48, 40, 5], [7, 7])]
DELTAS = np.array([-60, -20, 20, 60], np.int16)


def extreme_net(orc, seed, dims, shift, pair):
    """A net whose units change on a mid-grey image x, with the pair on every
    third unit of the last hidden layer and the label's bias set so that x
    keeps the label by a margin of half the domain's usual change; (net, x)."""
    g = I.rng(seed)
    net = I.random_qnet(g, dims, shift=shift, wmax=64, bmax=300)
    win = 128 << shift[0]
    net.b[0] = (g.uniform(0.0, 1.0, size=dims[1]) * win - net.W[0].astype(np.int64) @ np.full(dims[0], 128)).astype(np.int32)
    x = g.integers(112, 144, size=dims[0]).astype(np.uint8)
    label, other = 3, 1
    net.W[-1][other, ::3], net.W[-1][label, ::3] = pair
    z = orc.q8_forward(net, x)[0][-dims[-1]:].astype(np.int64)
    rest = np.delete(z, label)
    net.b[-1][label] += int(rest.max() - z[label] + 700)
    return net, x, label


@pytest.mark.parametrize("layers", range(len(DIMS)))
@pytest.mark.parametrize("pair", PAIRS)
def test_extreme_output_weights(orc, pair, layers):
    from paper_1907_12933_amd import ibmc
    dims, shift = DIMS[layers]
    net, x, label = extreme_net(orc, 40 + layers, dims, shift, pair)
    r = orc.q8_check(net, x, DELTAS, 1, 2, cap=1 << 21)
    assert r["clean_label"] == label and r["cex_total"] > 0
    ctx = ibmc.Context(0)
    m = ibmc.Mlp(ctx, net)
    for variant in (None, "fold"):
        ibmc.ibmc_set_variant(ctx, m, variant)
        s, cex, _ = ibmc.ibmc_check_property(ctx, m, x, DELTAS, 1, 2, cex_capacity=1 << 21)
        assert s["clean_label"] == r["clean_label"]
        assert list(s["cex"]) == [int(v) for v in r["cex"]]
        assert list(s["ties"]) == [int(v) for v in r["ties"]]
        assert np.array_equal(cex["k"], r["cex_k"]) and np.array_equal(cex["rank"], r["cex_rank"])
        assert np.array_equal(cex["new_label"], r["cex_label"])


@pytest.mark.parametrize("layers", range(len(DIMS)))
def test_lowest_weight_in_the_hidden_layers(orc, layers):
    """-128 in every layer: the joint bound of layers 1 and 2, whose absolute
    values must fit int8, is left out, and the intervals alone decide."""
    from paper_1907_12933_amd import ibmc
    dims, shift = DIMS[layers]
    net, x, _ = extreme_net(orc, 50 + layers, dims, shift, (64, -64))
    for W in net.W[:-1]:
        W[::2, ::3] = -128
    z = orc.q8_forward(net, x)[0][:dims[1]].astype(np.int64)
    net.b[0] += ((128 << shift[0]) // 2 - z).astype(np.int32)   # back into the window
    r = orc.q8_check(net, x, DELTAS, 1, 2, cap=1 << 21)
    ctx = ibmc.Context(0)
    m = ibmc.Mlp(ctx, net)
    ibmc.ibmc_set_variant(ctx, m, "fold")
    s, cex, _ = ibmc.ibmc_check_property(ctx, m, x, DELTAS, 1, 2, cex_capacity=1 << 21)
    assert r["cex_total"] > 0
    assert s["clean_label"] == r["clean_label"] and list(s["cex"]) == list(r["cex"]) and list(s["ties"]) == list(r["ties"])
    assert np.array_equal(cex["rank"], r["cex_rank"]) and np.array_equal(cex["new_label"], r["cex_label"])
