"""The FP32 lane enumeration at the class counts where its last layer changes
form (quads of class slots on the matrix cores: two, three or four, partly
filled or full), against the oracle's FP64 check; and clean potentials over
pixel counts around the load blocks of the clean pass.  Bar: the two
counterexample sets may differ only at points flagged as near ties."""
import numpy as np
import pytest

from paper_1907_12933_amd import inputs as I
from test_gpu_f32_instances import DELTAS, keys, make_net, near_boundary

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    from paper_1907_12933_amd import ibmc
    return ibmc.Context(0)


@pytest.mark.parametrize("n,h1,h2,nc", [
    (24, 16, 0, 2), (24, 64, 0, 8), (24, 64, 0, 9), (24, 128, 0, 12), (24, 32, 0, 13), (24, 128, 64, 3), (24, 64, 32, 9),
    (24, 128, 64, 12), (24, 128, 64, 13), (1, 16, 0, 3), (31, 64, 16, 5), (32, 16, 16, 4), (33, 128, 0, 4), (65, 100, 0, 10)])
def test_class_slots_and_clean_pass(ctx, orc, n, h1, h2, nc):
    from paper_1907_12933_amd import ibmc
    g = I.rng(40 * n + h1 + h2 + nc)
    net = make_net(g, [n, h1] + ([h2] if h2 else []) + [nc])
    x, top = near_boundary(net, g)
    m = ibmc.Mlp(ctx, net)
    k = min(n, 2)
    s, cex, ties = ibmc.ibmc_check_property(ctx, m, x, DELTAS, 1, k, near_tie_capacity=1 << 16)
    ref = orc.f64_check(net, x, DELTAS, 1, k, tie_rel=0.0)
    assert s["clean_label"] == top
    gpu, want = keys(cex["k"], cex["rank"]), keys(ref["cex_k"], ref["cex_rank"])
    flagged = keys(ties["k"], ties["rank"])
    assert gpu ^ want <= flagged
    assert len(flagged) <= max(10, len(want) // 10)
