"""A program that makes ordered searches and nothing else keeps its memory: the
pinned pieces that short record lists come back through are taken again on
every call, none are added."""
import numpy as np
import pytest

from paper_1907_12933_amd import inputs as I

pytestmark = pytest.mark.gpu


def mapped_bytes():
    with open("/proc/self/statm") as f:
        return int(f.read().split()[0]) * 4096


def test_many_short_ordered_searches():
    from paper_1907_12933_amd import ibmc
    g = I.rng(30)
    net = I.random_qnet(g, [16, 32, 24, 5], shift=[6, 6])
    x = g.integers(0, 255, size=(4, 16), endpoint=True).astype(np.uint8)[3]   # 208 counterexamples by the oracle
    D = np.array([-64, 64], np.int16)
    ctx = ibmc.Context(0)
    m, p = ibmc.Mlp(ctx, net), ibmc.Proposer(ctx, 3)

    def search():
        return ibmc.ibmc_check_property_ranked(ctx, m, p, x, 4, 4, D, 1, 2, cex_capacity=4096)

    first, recs = search()
    for _ in range(20):
        search()
    before = mapped_bytes()
    for _ in range(2000):
        s, r = search()
    # a piece is at least 512 bytes and often tens of KiB a call: 2,000 calls that
    # kept theirs would map 1 MiB in 256 KiB blocks at the least
    assert mapped_bytes() - before < 1 << 20
    assert s["cex"] == first["cex"] and np.array_equal(r, recs) and len(r) == 208
