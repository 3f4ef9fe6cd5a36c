"""GPU parity of the 32-passes-a-launch invasion against the oracle at its
edges: sides around one, two and three 64-site tiles, rows that start inside
a Philox call (L % 4 != 0), sources at a tile's corner, beside it and in the
lattice's corners, isolated and absent sources, media where the front dies
inside a launch, and dense media whose front crosses tiles in every
direction."""
import numpy as np
import pytest

from paper_cs_0312006_amd import workloads as W
from tests import gpu_util as G

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def b():
    from paper_cs_0312006_amd import binding
    binding.lib()
    return binding


@pytest.fixture(scope="module")
def o():
    from oracle import ref
    orc = ref.Oracle()
    orc.set_threads(G.host_threads())
    return orc


CASES = [
    W.Medium(2, 1.0, 1), W.Medium(31, 0.8, 2, 1, 30, 0), W.Medium(33, 0.7, 3, 1, 0, 32), W.Medium(66, 0.65, 4),
    W.Medium(127, 0.62, 5, 1, 63, 64), W.Medium(129, 0.9, 6, 1, 64, 63), W.Medium(191, 1.0, 7, 1, 190, 190),
    W.Medium(192, 0.95, 8, 1, 64, 64), W.Medium(193, 0.61, 9), W.Medium(254, 0.3, 10), W.Medium(320, 0.6, 11, 1, 159, 160),
    W.Medium(513, 0.6, 12), W.Medium(1030, 0.5927, 13), W.Medium(256, 0.5927, 14, 1, 128, 127),
]


@pytest.mark.parametrize("m", CASES, ids=lambda m: f"L{m.L}-P{m.porosity}-src{m.source}")
def test_invasion_equals_oracle(b, o, m):
    G.log(f"percolation {m}")
    ctx = b.perc_create(m.L, m.porosity, m.seed, m.source, m.i0, m.j0)
    try:
        b.perc_run(ctx)
        r = b.perc_result_get(ctx)
        pore, arr = b.perc_copy_medium(ctx, m.L), b.perc_copy_arrival(ctx, m.L)
    finally:
        b.perc_destroy(ctx)
    pore_o = o.perc_medium(m.L, m.porosity, m.seed)
    assert np.array_equal(pore, pore_o), "medium differs"
    arr_o = o.perc_invade(pore_o, m.source, m.i0, m.j0)
    assert np.array_equal(arr, arr_o), f"first {np.argwhere(arr != arr_o)[:5].tolist()}"
    inv, mx, sp = o.perc_summary(arr_o)
    assert (r.pores, r.invaded, r.passes, r.spans) == (int(pore_o.sum()), inv, mx, sp)


def test_batches_of_growing_size_share_a_context(b, o):
    """The first context of a batch keeps the batch's table and lists: runs
    alone and in batches of one, three and two media, in any order, agree
    with the oracle."""
    media = [W.Medium(200, 0.62, 31), W.Medium(65, 0.7, 32, 1, 10, 60), W.Medium(300, 0.6, 33)]
    want = [o.perc_invade(o.perc_medium(m.L, m.porosity, m.seed), m.source, m.i0, m.j0) for m in media]
    ctxs = [b.perc_create(m.L, m.porosity, m.seed, m.source, m.i0, m.j0) for m in media]
    try:
        for group in ([0], [1, 0, 2], [1], [0, 2], [2, 1]):
            G.log(f"percolation batch {group}")
            b.perc_run_batch([ctxs[k] for k in group])
            for k in group:
                assert np.array_equal(b.perc_copy_arrival(ctxs[k], media[k].L), want[k]), (group, k)
        b.perc_run(ctxs[1])
        assert np.array_equal(b.perc_copy_arrival(ctxs[1], media[1].L), want[1])
    finally:
        for c in ctxs:
            b.perc_destroy(c)
