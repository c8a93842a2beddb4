"""stop_at_first with records that stay on the device: the levels' records are
gathered on the host, level by level, and sent to the caller's device buffer;
they are those of the same call with host buffers, for lists that one
workgroup sorts (up to 4,096 slots) and longer ones, and for near ties."""
import numpy as np
import pytest

from paper_1907_12933_amd import inputs as I

pytestmark = pytest.mark.gpu


def both(ibmc, ctx, props, **kw):
    import torch
    host = ibmc.ibmc_check_batch(ctx, props, stop_at_first=True, **kw)
    buf = torch.zeros((kw["cex_capacity"] + 1) * ibmc.CEX_DTYPE.itemsize, dtype=torch.uint8, device="cuda")
    dev = ibmc.ibmc_check_batch(ctx, props, stop_at_first=True, records_on_device=True, cex_buf=buf, **kw)
    assert [(s["clean_label"], s["levels"], s["cex"], s["ties"]) for s in dev[0]] == \
        [(s["clean_label"], s["levels"], s["cex"], s["ties"]) for s in host[0]] and dev[3] == host[3]
    cex = np.frombuffer(dev[1].cpu().numpy().tobytes(), ibmc.CEX_DTYPE)
    assert np.array_equal(cex, host[1])
    ties = np.frombuffer(dev[2].cpu().numpy().tobytes(), ibmc.CEX_DTYPE)
    assert np.array_equal(ties, host[2])
    return host


@pytest.mark.parametrize("deltas,least", [([-96, 96], 1), (list(range(-96, 97, 8)), 4097)])
def test_integer_records(orc, deltas, least):
    from paper_1907_12933_amd import ibmc
    ctx = ibmc.Context(0)
    g = I.rng(7)
    D = np.array(deltas, np.int16)
    while True:   # none at level 1, some at a later one, by the oracle
        net = I.random_qnet(g, [24, 40, 5], shift=4, wmax=12, bmax=100)
        X = g.integers(0, 255, size=(2, 24), endpoint=True).astype(np.uint8)
        r = [orc.q8_check(net, x, D, 1, 2, cap=1 << 20, stop_at_first=True) for x in X]
        if r[0]["cex"][0] == 0 and sum(q["cex_total"] for q in r) >= least:
            break
    m = ibmc.Mlp(ctx, net)
    for cap in (1 << 18, least // 2 + 1):
        sums, cex, _, _ = both(ibmc, ctx, [(m, x, D, 1, 2) for x in X], cex_capacity=cap)
        for i, q in enumerate(r):
            assert list(sums[i]["cex"]) == list(q["cex"])
            if cap == 1 << 18:
                assert np.array_equal(cex["rank"][cex["prop"] == i], q["cex_rank"])


def test_near_ties():
    from paper_1907_12933_amd import ibmc
    ctx = ibmc.Context(0)
    g = I.rng(11)
    m = ibmc.Mlp(ctx, I.random_fnet(g, [24, 32, 16, 5], scale=2.0))
    x = g.integers(0, 255, size=24, endpoint=True).astype(np.uint8)
    # every point is a near tie
    host = both(ibmc, ctx, [(m, x, np.array([-8, 8], np.int16), 1, 2)], cex_capacity=1 << 12, near_tie_capacity=1 << 12,
                near_tie_rel=1e9)
    assert len(host[2]) == 48 + 1104
