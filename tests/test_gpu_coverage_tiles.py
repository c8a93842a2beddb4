"""Coverage of input pairs at the edges of the pair kernel's tiles: 16 and 32
pairs a workgroup with remainders (4,129 pairs take the larger tile), rows of
pixels loaded whole (a multiple of sixteen) or byte by byte, layers whose
16-row tiles do not split evenly over the sixteen waves, potentials and ratios
within and beyond the 24-bit tests, against the oracle.  All-integer, so
equality is exact."""
import numpy as np
import pytest

from paper_1907_12933_amd import inputs as I
from test_gpu_coverage import CRITS, same

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    from paper_1907_12933_amd import ibmc
    return ibmc.Context(0)


def potentials(net, X):
    a, out = X.astype(np.int64), []
    for l, (w, b) in enumerate(zip(net.W, net.b)):
        u = a @ w.astype(np.int64).T + b.astype(np.int64)
        out.append(u)
        if l < len(net.W) - 1:
            a = np.clip(u >> net.shift[l], 0, 127)
    return np.concatenate(out, 1)


# (dims, shift, largest weight, pairs, ratio terms)
CASES = [
    ([16, 48, 20, 7], 5, 20, 4129, (3, 2)),
    ([30, 16, 33, 5], 4, 20, 4097, (3, 2)),
    ([64, 272, 130, 3], 6, 20, 33, (3, 2)),
    ([48, 600, 1024, 9], 7, 30, 17, (5, 1)),
    ([784, 900, 40, 7], 10, 127, 40, (3, 2)),        # potentials beyond 2^24
    ([400, 64, 64, 10], 9, 127, 32, (70000, 60000)),  # products beyond 2^32
    ([400, 64, 64, 10], 9, 127, 1, (20000000, 3)),    # a ratio beyond 2^24
]


@pytest.mark.parametrize("dims,shift,wmax,pairs,ratio", CASES)
def test_pair_tiles(ctx, orc, dims, shift, wmax, pairs, ratio):
    import torch
    from paper_1907_12933_amd import ibmc
    g = I.rng(sum(dims) + pairs)
    net = I.random_qnet(g, dims, shift=shift, wmax=wmax, bmax=300)
    if wmax == 127:
        net.W[0][:3] = [[127], [-127], [64]]
    x1 = g.integers(0, 255, size=(pairs, dims[0]), endpoint=True).astype(np.uint8)
    x2 = np.stack([I.perturbed_partner(g, x, 6, 60) for x in x1])
    x2[::5] = x1[::5]
    x2[1::7] = 255 - x1[1::7]
    P1, P2 = potentials(net, x1), potentials(net, x2)
    m = ibmc.Mlp(ctx, net)
    opt = dict(dist_sq_min=50, ratio_num=ratio[0], ratio_den=ratio[1])
    outs = ibmc.ibmc_coverage_all_dev(ctx, m, torch.from_numpy(x1).cuda(), torch.from_numpy(x2).cuda(), **opt)
    for c, got in zip(CRITS, outs):
        ref = orc.coverage(dims[1:], P1, P2, c, **opt)
        same(got, ref)
        same(ibmc.ibmc_coverage(ctx, m, x1, x2, c, **opt), ref)
    # images at an odd address
    pad = torch.zeros(2, pairs * dims[0] + 1, dtype=torch.uint8, device="cuda")
    pad[0, 1:] = torch.from_numpy(x1).cuda().flatten()
    pad[1, 1:] = torch.from_numpy(x2).cuda().flatten()
    again = ibmc.ibmc_coverage_all_dev(ctx, m, pad[0, 1:].view(pairs, -1), pad[1, 1:].view(pairs, -1), **opt)
    for a, b in zip(outs, again):
        assert np.array_equal(a["bits"], b["bits"]) and a["covered_neurons"] == b["covered_neurons"]
