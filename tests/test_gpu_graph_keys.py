"""The kept graph of a multi-network batch is replayed only for a batch whose
captured launches would be the same.  Two networks whose units are nearly all
live are scanned for folding (from 30,000 points of a call on) and not folded:
the scan has done their clean pass, so the captured graph holds none, and a
batch of the same plans that is not scanned must not replay it."""
import numpy as np
import pytest

from paper_1907_12933_amd import inputs as I

pytestmark = pytest.mark.gpu

DIMS = [20, 100, 10]
PER_NET = 47


def all_live_net(seed):
    """Every first-layer potential of a mid-grey image inside the requantiser's window."""
    g = I.rng(seed)
    net = I.random_qnet(g, DIMS, shift=[6], wmax=64, bmax=300)
    c = g.uniform(0.2, 0.8, size=DIMS[1]) * (128 << 6)
    net.b[0] = (c - net.W[0].astype(np.int64) @ np.full(DIMS[0], 128)).astype(np.int32)
    return net


def batch(ibmc, ctx, orc, nets, ms, seed, D):
    """One batch over both networks with images of its own, against the oracle."""
    g = I.rng(seed)
    X = g.integers(112, 144, size=(2 * PER_NET, DIMS[0])).astype(np.uint8)
    sums, recs, _, rc = ibmc.ibmc_check_batch(ctx, [(ms[i // PER_NET], X[i], D, 1, 1) for i in range(len(X))])
    assert rc == ibmc.IBMC_OK
    total = 0
    for i, x in enumerate(X):
        r = orc.q8_check(nets[i // PER_NET], x, D, 1, 1)
        assert sums[i]["clean_label"] == r["clean_label"], i
        assert list(sums[i]["cex"]) == list(r["cex"]) and list(sums[i]["ties"]) == list(r["ties"]), i
        c = recs[recs["prop"] == i]
        assert np.array_equal(c["rank"], r["cex_rank"]) and np.array_equal(c["new_label"], r["cex_label"]), i
        total += r["cex_total"]
    assert total > 0


@pytest.mark.parametrize("scanned_first", [True, False])
@pytest.mark.parametrize("how", ["points", "variant"])
def test_scanned_and_unscanned_batches(orc, how, scanned_first):
    from paper_1907_12933_amd import ibmc
    ctx = ibmc.Context(0)
    nets = [all_live_net(60), all_live_net(61)]
    ms = [ibmc.Mlp(ctx, n) for n in nets]
    # 94 properties of 320 points are scanned, of 300 (as many chunks) are not
    wide = np.array([d for d in range(-64, 65, 8) if d], np.int16)
    assert wide.size == 16
    names = [ibmc.ibmc_chosen_variant(ctx, m) for m in ms]
    for step in range(4):
        scanned = (step % 2 == 0) == scanned_first
        D = wide
        if how == "points":
            D = wide if scanned else np.delete(wide, 5)
        else:
            for m, name in zip(ms, names):
                ibmc.ibmc_set_variant(ctx, m, None if scanned else name)
        batch(ibmc, ctx, orc, nets, ms, 80 + step, D)
    launches, _ = ibmc.ibmc_graph_stats(ctx)
    assert launches == 4   # nothing was folded
