"""The FP32 enumeration of wide networks, whose sixteen points are shared by a
wave per 64 units of the widest layer: one to eight waves, layers narrower and
wider than others, two to four weight layers, point counts that end inside a
chunk, against the oracle's FP64 check.  Bar: the two counterexample sets may
differ only at points flagged as near ties."""
import numpy as np
import pytest

from paper_1907_12933_amd import inputs as I
from test_gpu_f32_instances import DELTAS, keys, make_net, near_boundary

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    from paper_1907_12933_amd import ibmc
    return ibmc.Context(0)


@pytest.mark.parametrize("dims,k", [
    ([9, 30, 20], 2), ([13, 129, 7], 2), ([10, 64, 65, 4], 2), ([11, 200, 60, 5], 2), ([9, 40, 300, 6], 2),
    ([8, 512, 33, 3], 2), ([7, 65, 448, 128, 9], 2), ([17, 384, 384, 10], 1)])
def test_wide_float_checks(ctx, orc, dims, k):
    from paper_1907_12933_amd import ibmc
    g = I.rng(sum(dims))
    net = make_net(g, dims)
    x, top = near_boundary(net, g)
    m = ibmc.Mlp(ctx, net)
    print(dims, flush=True)
    s, cex, ties = ibmc.ibmc_check_property(ctx, m, x, DELTAS, 0, k, near_tie_capacity=1 << 16)
    ref = orc.f64_check(net, x, DELTAS, 0, k, tie_rel=0.0)
    assert s["clean_label"] == top and list(s["points"]) == [int(v) for v in ref["points"]]
    gpu, want = keys(cex["k"], cex["rank"]), keys(ref["cex_k"], ref["cex_rank"])
    flagged = keys(ties["k"], ties["rank"])
    assert gpu ^ want <= flagged
    assert len(flagged) <= max(10, len(want) // 10)
