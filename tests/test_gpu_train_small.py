"""Training of small networks: sample counts around the sixteen rows that one
thread of the weights kernel stages and the sixteen samples of a running sum,
and the pass's rows kept in the context, which networks of other sizes have
used before: gradients and losses against FP64, bit-equal to a context's first."""
import numpy as np
import pytest

from paper_1907_12933_amd import inputs as I

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    from paper_1907_12933_amd import ibmc
    return ibmc.Context(0)


def draw(g, dims, n):
    net = I.random_fnet(g, dims, scale=2.0)
    net.b = [(g.standard_normal(d) * 0.5).astype(np.float32) for d in dims[1:]]
    imgs = g.integers(0, 255, size=(n, dims[0]), endpoint=True).astype(np.uint8)
    labs = g.integers(0, dims[-1] - 1, size=n, endpoint=True).astype(np.int32)
    return net, imgs, labs


# FP32 sums of at most ~260 terms against FP64: below 260 * 2^-24 = 1.6e-5 of the
# sum of magnitudes, at most 7e-5 of the largest entry as in the tile tests
@pytest.mark.parametrize("n", [1, 15, 16, 17, 33, 241, 256, 257, 1041])
def test_sample_counts(ctx, orc, n):
    from paper_1907_12933_amd import ibmc
    net, imgs, labs = draw(I.rng(500 + n), [35, 16, 5], n)
    loss, grad = ibmc.ibmc_mlp_loss_grad(ctx, ibmc.Mlp(ctx, net), imgs, labs)
    rl, rg = orc.f64_loss_grad(net, imgs, labs)
    assert loss == pytest.approx(rl, rel=1e-5)
    assert np.max(np.abs(grad - rg)) <= 7e-5 * np.max(np.abs(rg))
    # one step per batch, the last one smaller
    other = ibmc.Context(0)
    fits = []
    for c in (ctx, other):
        t, l = ibmc.ibmc_fit_mlp(c, ibmc.Mlp(c, net), imgs, labs, epochs=2, batch=15)
        fits.append(([w.tobytes() for w in t.params[0] + t.params[1]], l.tobytes()))
    assert fits[0] == fits[1]


def test_rows_of_other_networks(ctx):
    from paper_1907_12933_amd import ibmc
    g = I.rng(560)
    cases = [draw(g, d, n) for d, n in (([35, 16, 5], 900), ([100, 64, 48, 10], 3000), ([784, 32, 10], 4000), ([20, 8, 3], 17))]
    for net, imgs, labs in cases + cases[::-1]:
        fresh = ibmc.Context(0)
        l0, g0 = ibmc.ibmc_mlp_loss_grad(fresh, ibmc.Mlp(fresh, net), imgs, labs)
        l1, g1 = ibmc.ibmc_mlp_loss_grad(ctx, ibmc.Mlp(ctx, net), imgs, labs)
        assert l0 == l1 and np.array_equal(g0, g1)
