"""GPU parity of the Creutz band kernel (a wave per row, demons in registers)
against the oracle: rows that fill, end inside and start inside a wave's
words, bands with and without rows outside them, forward and reversed calls
of every length (one and two sweeps run on the streaming kernels), demons up
to the cap of 255, exact return, and Metropolis sweeps in between."""
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


# L, largest demon, calls (negative: reversed sweeps)
CASES = [
    (4, 3, [5, -3]), (6, 255, [4]), (10, 2, [3, -4, 7]), (16, 255, [9, -2, 6]), (34, 4, [7, 1, 5]),
    (66, 255, [40, -35]), (72, 3, [6, 2, -6]), (250, 6, [5, -3]), (508, 3, [4]), (512, 4, [33, -5, 1]),
    (520, 255, [4, -4]), (1000, 3, [6]), (1002, 5, [3, -3, 2]), (1024, 255, [9, -9]), (1536, 2, [4]),
    (2048, 3, [5, -3]), (2050, 3, [3]), (2560, 4, [3, -3]), (3080, 3, [3]), (3584, 3, [-3]), (4086, 2, [3]),
    (4096, 3, [4, -3]),
]


@pytest.mark.parametrize("L,hi,calls", CASES)
def test_creutz_rows_equal_oracle(b, o, L, hi, calls):
    d = W.random_demons(L, 100 + L, hi)
    ctx = b.ising_create(L, 1.0, 0.0, 2.0, 40 + L, 0.6)
    try:
        b.ising_creutz_init(ctx, d)
        s = o.init(L, 40 + L, 0.6)
        for n in calls:
            G.log(f"creutz L={L} hi={hi} n={n}")
            b.ising_creutz_sweep(ctx, abs(n), n < 0)
            _, B, M = b.ising_observables(ctx, b.ISING_OBS_SERIES)
            Bo, Mo, Do = o.creutz_run(s, d, abs(n), reverse=n < 0)
            assert np.array_equal(B, Bo) and np.array_equal(M, Mo), (L, n)
        assert np.array_equal(b.ising_copy_spins(ctx, L), s)
        assert np.array_equal(b.ising_copy_demons(ctx, L), d)
    finally:
        b.ising_destroy(ctx)


def test_long_runs_return_and_mix_with_metropolis(b, o):
    """600 sweeps (two launches) and 600 reversed ones restore the lattice
    and the demons; Metropolis sweeps of the same context in between use the
    same edge slots."""
    L = 200
    d = W.random_demons(L, 9, 5)
    ctx = b.ising_create(L, 1.0, 0.0, 2.3, 77, 0.5)
    try:
        b.ising_creutz_init(ctx, d)
        start = b.ising_copy_spins(ctx, L)
        G.log("creutz 600 and back")
        b.ising_creutz_sweep(ctx, 600)
        b.ising_creutz_sweep(ctx, 600, True)
        assert np.array_equal(b.ising_copy_spins(ctx, L), start) and np.array_equal(b.ising_copy_demons(ctx, L), d)
        b.ising_observables(ctx, b.ISING_OBS_SERIES)
        G.log("metropolis, creutz, metropolis")
        b.ising_sweep(ctx, 30)
        b.ising_creutz_sweep(ctx, 20)
        b.ising_sweep(ctx, 5)
        s = o.init(L, 77, 0.5)
        o.run(s, 1.0, 0.0, 2.3, 77, 0, 30)
        o.creutz_run(s, d, 20)
        o.run(s, 1.0, 0.0, 2.3, 77, 30, 5)
        assert np.array_equal(b.ising_copy_spins(ctx, L), s) and np.array_equal(b.ising_copy_demons(ctx, L), d)
    finally:
        b.ising_destroy(ctx)
