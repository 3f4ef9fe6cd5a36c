"""Sweeps over wave tiles of any row length: the sides and tables they serve
(beyond 4096 in a field, beyond 16384 without) against the per-site plan on
the same runs and against the oracle on windows across the periodic edge and
between two tiles. Last columns of one word, of one whole lane, of part of a
lane, and none; last bands of 8 and of 16 rows; even and odd sweeps."""
import numpy as np
import pytest

from oracle import ref
from tests import gpu_util as G

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def b():
    from paper_cs_0312006_amd import binding
    binding.lib()
    return binding


def _run(b, L, calls, **p):
    c = b.ising_create(L, **p)
    try:
        for n in calls:
            b.ising_sweep(c, n)
        obs, B, M = b.ising_observables(c, b.ISING_OBS_SERIES)
        return B, M, b.ising_copy_spins(c, L), obs
    finally:
        b.ising_destroy(c)


@pytest.mark.parametrize("L,J,h,T,calls", [
    (4104, 1.0, 0.1, 2.3, (5,)),      # two words a lane, 8-row tiles, a last column of one word
    (4112, -1.0, 0.1, 2.3, (1, 2)),   # of one lane
    (6136, 1.0, -0.3, 1.0, (4,)),     # a last lane of one word, 63 lanes whole
    (8192, 1.0, 0.1, 0.05, (2,)),     # whole columns, 16-row tiles; zero and certain thresholds
    (8200, 1.0, 0.1, 2.3, (3, 2)),    # a last band of 8 rows
    (16392, 1.0, 0.0, 2.3, (3,)),     # four words a lane, the last column one word
    (18432, 1.0, 0.0, 2.3, (2,)),     # whole columns: the fused tiles, in place of full rows
    (20024, 1.0, 0.0, 0.05, (2,)),    # three words of the last lane
    (32760, 1.0, 0.2, 2.3, (2,)),
])
def test_tiles_match_the_per_site_plan_and_the_oracle(b, L, J, h, T, calls):
    o, n = ref.default(), sum(calls)
    p = dict(J=J, h=h, T=T, seed=0x1234567890 + L, p_up=0.4)
    G.log(f"tiles L={L} J={J} h={h} T={T} calls={calls}")
    B, M, s, obs = _run(b, L, calls, **p)
    B1, M1, s1, _ = _run(b, L, (n,), flags=b.ISING_PLAN_GENERIC, **p)
    assert len(B) == n and np.array_equal(B, B1) and np.array_equal(M, M1) and np.array_equal(s, s1)
    assert (obs.bond_sum, obs.mag_sum) == (B[-1], M[-1]) and M[-1] == s.sum(dtype=np.int64)
    wide = 4 * n + 40
    for i0, j0 in ((L - wide // 2, L - wide // 2), (L // 2 - 20, 64 * 8 * 4 - wide // 2)):
        win = o.init_window(L, p["seed"], p["p_up"], i0, j0, wide)
        win, valid = o.window_run(L, J, h, T, p["seed"], 0, n, i0, j0, win)
        got = s[np.ix_((np.arange(wide) + i0) % L, (np.arange(wide) + j0) % L)]
        assert valid.any() and np.array_equal(got[valid], win[valid])
