"""The kept graph of a multi-network batch holds its networks' layouts (weights'
addresses, shifts), so it belongs to the networks loaded, not to the places
where their handles lie: after they are freed, others of the same shapes, which
may get the same addresses, must have a graph of their own."""
import numpy as np
import pytest

from paper_1907_12933_amd import inputs as I

pytestmark = pytest.mark.gpu


def test_networks_loaded_in_the_place_of_freed_ones(orc):
    from paper_1907_12933_amd import ibmc
    ctx = ibmc.Context(0)
    D = np.array([-60, -20, 20, 60], np.int16)
    g = I.rng(90)
    for step in range(6):
        nets = [I.random_qnet(g, [30, 40, 6], shift=5 + step % 3), I.random_qnet(g, [24, 64, 32, 5], shift=[6, 4 + step % 3])]
        ms = [ibmc.Mlp(ctx, n) for n in nets]
        X = [g.integers(0, 255, size=n.dims[0], endpoint=True).astype(np.uint8) for n in nets]
        refs = [orc.q8_check(n, x, D, 1, 2, cap=1 << 20) for n, x in zip(nets, X)]
        for again in range(2):
            sums, recs, _, _ = ibmc.ibmc_check_batch(ctx, [(m, x, D, 1, 2) for m, x in zip(ms, X)])
            for i, r in enumerate(refs):
                assert sums[i]["clean_label"] == r["clean_label"] and list(sums[i]["cex"]) == list(r["cex"]), (step, i)
                c = recs[recs["prop"] == i]
                assert np.array_equal(c["rank"], r["cex_rank"]) and np.array_equal(c["new_label"], r["cex_label"])
            launches, reuses = ibmc.ibmc_graph_stats(ctx)
            assert (launches, reuses) == (2 * step + again + 1, step + again)
        for m in ms:
            m.close()
