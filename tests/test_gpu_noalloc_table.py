"""The table sigmoid through the allocation-free entry point: its table lies in
the fixed scratch for that call only, so what later calls put there must not
change a later table check (Sec. IV-D's table, FP32)."""
import numpy as np
import pytest

from paper_1907_12933_amd import inputs as I

pytestmark = pytest.mark.gpu


def test_table_check_after_the_scratch_was_used_again(orc):
    from paper_1907_12933_amd import ibmc
    g = I.rng(17)
    D = np.array([-96, -48, 48, 96], np.int16)
    qnet = I.random_qnet(g, [24, 40, 5], shift=4, wmax=12, bmax=100)
    while True:   # the first drawn network and image with counterexamples by the oracle
        fnet = I.random_fnet(g, [24, 32, 16, 5], scale=4.0)
        x = g.integers(0, 255, size=24, endpoint=True).astype(np.uint8)
        if orc.f64_check(fnet, x, D, 1, 2, lut=True)["cex_total"] > 10:
            break

    def table(ctx, m, entry):
        s, cex, ties = ibmc.ibmc_check_property(ctx, m, x, D, 1, 2, cex_capacity=1 << 14, near_tie_capacity=1 << 14,
                                                table_sigmoid=True, _entry=entry)
        return s["clean_label"], s["cex"], s["ties"], cex.tobytes(), ties.tobytes()

    other = ibmc.Context(0)
    want = table(other, ibmc.Mlp(other, fnet), "ibmc_check_property")
    assert sum(want[1]) > 10
    ctx = ibmc.Context(0)
    fm, qm = ibmc.Mlp(ctx, fnet), ibmc.Mlp(ctx, qnet)
    for entry in ("ibmc_check_property_noalloc", "ibmc_check_property", "ibmc_check_property_noalloc"):
        assert table(ctx, fm, entry) == want, entry
        # records over the scratch's first megabytes
        s, _, _ = ibmc.ibmc_check_property_noalloc(ctx, qm, x, np.arange(-96, 97, 16), 1, 3, cex_capacity=1 << 19)
        assert s["cex_total"] > 1 << 17
