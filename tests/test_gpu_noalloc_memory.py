"""The allocation-free check allocates and frees nothing: the process's mappings
of 128 KiB and more are the same before and after a context's first such call
(record lists of both sorts, short and radix, and levels after each other) and
after one that follows plain checks, which leave several staging blocks; the
results are the oracle's."""
import numpy as np
import pytest

from paper_1907_12933_amd import inputs as I

pytestmark = pytest.mark.gpu


# (deltas, k_max, stop_at_first, least and most records by the oracle)
CASES = {
    "short": ([-96, -48, 48, 96], 1, False, 1, 4096),
    "long": (list(range(-96, 97, 16)), 2, False, 4097, 1 << 15),
    "levels": ([-96, 96], 3, True, 1, 4096),
}


def drawn(orc, case):
    """The first drawn network and image with as many records as the case asks
    for (and none at level 1 where levels follow each other)."""
    deltas, k, stop, least, most = CASES[case]
    D = np.array(deltas, np.int16)
    g = I.rng(7)
    while True:
        net = I.random_qnet(g, [24, 40, 5], shift=4, wmax=12, bmax=100)
        x = g.integers(0, 255, size=24, endpoint=True).astype(np.uint8)
        r = orc.q8_check(net, x, D, 1, k, cap=1 << 20, stop_at_first=stop)
        if least <= r["cex_total"] <= most and (not stop or r["cex"][0] == 0):
            return net, x, D, r


def mappings():
    found = set()
    with open("/proc/self/maps") as f:
        for line in f:
            lo, hi = (int(v, 16) for v in line.split()[0].split("-"))
            if hi - lo >= 128 << 10 and "[heap]" not in line:
                found.add((lo, hi))
    return found


@pytest.mark.parametrize("after_plain", [False, True])
@pytest.mark.parametrize("case", sorted(CASES))
def test_the_call_maps_and_unmaps_nothing(orc, case, after_plain):
    from paper_1907_12933_amd import ibmc
    net, x, D, r = drawn(orc, case)
    k, stop = CASES[case][1:3]
    # (kernels are loaded and the runtime's own buffers made by an earlier context)
    warm = ibmc.Context(0)
    wm = ibmc.Mlp(warm, net)
    ibmc.ibmc_check_property_noalloc(warm, wm, x, D, 1, k, stop_at_first=stop, cex_capacity=1 << 15)
    ctx = ibmc.Context(0)
    m = ibmc.Mlp(ctx, net)
    if after_plain:
        # 3,000 properties: more staging than the first block holds
        ibmc.ibmc_check_batch(ctx, [(m, x, D, 1, 1)] * 3000, cex_capacity=1 << 16)
    cex = np.zeros(1 << 15, ibmc.CEX_DTYPE)
    o = ibmc._opts(1, k, 1, stop, len(cex), 0, 0.0)
    s = ibmc.ibmc_check_summary()
    args = (ctx.handle, m.handle, ibmc._ptr(x, ibmc.P_U8), x.size, ibmc._ptr(D, ibmc.P_I16), D.size, ibmc.C.byref(o),
            ibmc.C.byref(s), cex.ctypes.data_as(ibmc.P_CEX), None)
    call = ibmc.lib().ibmc_check_property_noalloc
    before = mappings()
    rc = call(*args)
    after = mappings()
    assert rc == ibmc.IBMC_OK
    assert before == after, (before - after, after - before)
    d = ibmc.summary_dict(s)
    assert d["clean_label"] == r["clean_label"] and list(d["cex"]) == list(r["cex"])
    n = int(r["cex_total"])
    assert np.array_equal(cex["rank"][:n], r["cex_rank"]) and np.array_equal(cex["new_label"][:n], r["cex_label"])
