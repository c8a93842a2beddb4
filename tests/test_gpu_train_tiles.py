"""GPU gradient of the float networks at the edges of the training kernels'
tiles: layer widths around 16 (weight tiles), 64 (row blocks of the pass) and
multiples of four (input steps), sample counts around four (samples per
workgroup), and a set larger than one pass."""
import numpy as np
import pytest

from paper_1907_12933_amd import inputs as I

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    from paper_1907_12933_amd import ibmc
    return ibmc.Context(0)


# FP32 sums of at most ~1,100 terms against FP64: relative rounding of a sum is
# below terms * 2^-24 of the sum of magnitudes, at most 7e-5 of the largest entry
@pytest.mark.parametrize("dims,n", [([15, 16, 17, 2], 4), ([16, 63, 64, 3], 5), ([17, 65, 15, 16], 3), ([3, 64, 5], 1),
                                    ([64, 4, 129, 17], 66), ([33, 1024, 65, 64], 7), ([1024, 18, 33, 10, 12], 258)])
def test_gradient_at_tile_edges(ctx, orc, dims, n):
    from paper_1907_12933_amd import ibmc
    g = I.rng(sum(dims) + n)
    net = I.random_fnet(g, dims, scale=2.0)
    net.b = [(g.standard_normal(d) * 0.5).astype(np.float32) for d in dims[1:]]
    imgs = g.integers(0, 255, size=(n, dims[0]), endpoint=True).astype(np.uint8)
    labs = g.integers(0, dims[-1] - 1, size=n, endpoint=True).astype(np.int32)
    loss, grad = ibmc.ibmc_mlp_loss_grad(ctx, ibmc.Mlp(ctx, net), imgs, labs)
    rl, rg = orc.f64_loss_grad(net, imgs, labs)
    assert loss == pytest.approx(rl, rel=1e-5)
    assert np.max(np.abs(grad - rg)) <= 7e-5 * np.max(np.abs(rg))


def test_a_set_of_two_passes_equals_its_parts(ctx):
    """40,000 samples of a 1,000-pixel net take two passes (256 MiB of rows);
    the mean gradient and loss equal those of its halves, each one pass."""
    from paper_1907_12933_amd import ibmc
    g = I.rng(77)
    net = I.random_fnet(g, [1000, 24, 10])
    imgs = g.integers(0, 255, size=(40000, 1000), endpoint=True).astype(np.uint8)
    labs = g.integers(0, 9, size=40000, endpoint=True).astype(np.int32)
    m = ibmc.Mlp(ctx, net)
    loss, grad = ibmc.ibmc_mlp_loss_grad(ctx, m, imgs, labs)
    parts = [ibmc.ibmc_mlp_loss_grad(ctx, m, imgs[s], labs[s]) for s in (slice(0, 20000), slice(20000, 40000))]
    assert loss == pytest.approx(sum(p[0] for p in parts) / 2, rel=1e-6)
    ref = (parts[0][1].astype(np.float64) + parts[1][1]) / 2
    # sums of 40,000 terms in blocks of 64: rounding well below 1e-5 of the largest entry
    assert np.max(np.abs(grad - ref)) <= 1e-5 * np.max(np.abs(ref))
