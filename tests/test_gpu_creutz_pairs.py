"""GPU parity of the two-sweeps-a-launch Creutz kernel against the oracle:
sides beyond the bands whose rows fill the waves, end inside a lane's words
and inside a wave, bands whose last one is short, forward and reversed calls
of odd and even length, demons up to 255, at each number of words a lane."""
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
CASES = [(4104, 255, [2, -2, 3]), (4352, 3, [5, -4]), (5000, 4, [2, -3]), (8192, 3, [3, -2]), (8200, 255, [2]),
         (10000, 3, [-2, 2]), (16384, 3, [2]), (16392, 3, [-2]), (20016, 4, [2])]


@pytest.mark.parametrize("L,hi,calls", CASES)
def test_creutz_pairs_equal_oracle(b, o, L, hi, calls):
    d = W.random_demons(L, 100 + L, hi)
    ctx = b.ising_create(L, 1.0, 0.0, 2.0, 40 + L, 0.6)
    try:
        b.ising_creutz_init(ctx, d)
        s = o.init(L, 40 + L, 0.6)
        for n in calls:
            G.log(f"creutz pairs L={L} hi={hi} n={n}")
            b.ising_creutz_sweep(ctx, abs(n), n < 0)
            _, B, M = b.ising_observables(ctx, b.ISING_OBS_SERIES)
            Bo, Mo, _ = o.creutz_run(s, d, abs(n), reverse=n < 0)
            assert np.array_equal(B, Bo) and np.array_equal(M, Mo), (L, n)
        assert np.array_equal(b.ising_copy_spins(ctx, L), s)
        assert np.array_equal(b.ising_copy_demons(ctx, L), d)
    finally:
        b.ising_destroy(ctx)
