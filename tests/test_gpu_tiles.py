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
    (12296, 1.0, 0.1, 2.3, (2,)),     # buffers beyond the cache
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


def test_stepped_batches_beyond_and_within_the_cache(b):
    """The same lattices stepped in one batch of 302 MB (both buffers) and in
    two of 67 and 235 MB."""
    sides = [4096] * 2 + [4096, 4080, 4064, 4096, 4048, 4096, 4032]
    G.log("stepped batches around the cache's size")
    one = [b.ising_create(L, h=0.02, T=2.3, seed=L + k) for k, L in enumerate(sides)]
    two = [b.ising_create(L, h=0.02, T=2.3, seed=L + k) for k, L in enumerate(sides)]
    try:
        b.ising_sweep_batch_plan(one, [3] * 9, b.ISING_BATCH_STEPPED)
        for part in (two[:2], two[2:]):
            b.ising_sweep_batch_plan(part, [3] * len(part), b.ISING_BATCH_STEPPED)
        for k, L in enumerate(sides):
            (_, B, M), (_, B2, M2) = (b.ising_observables(c[k], b.ISING_OBS_SERIES) for c in (one, two))
            assert np.array_equal(B, B2) and np.array_equal(M, M2)
            assert np.array_equal(b.ising_copy_spins(one[k], L), b.ising_copy_spins(two[k], L))
        r = b.ising_create(sides[3], h=0.02, T=2.3, seed=sides[3] + 3)
        try:
            b.ising_sweep(r, 3)
            assert np.array_equal(b.ising_copy_spins(r, sides[3]), b.ising_copy_spins(one[3], sides[3]))
        finally:
            b.ising_destroy(r)
    finally:
        for c in one + two:
            b.ising_destroy(c)


@pytest.mark.parametrize("L,h,creutz", [(4104, 0.1, False), (4104, 0.0, True)])
def test_captured_sweeps_stay_valid(b, L, h, creutz):
    """A graph of static sweeps holds the lattice's address: odd tile sweeps
    and reversed Creutz pairs leave the lattice where it was."""
    import torch
    G.log(f"graph after eager sweeps L={L} creutz={creutz}")
    s, n = torch.cuda.Stream(), 2
    p = dict(J=1.0, h=h, T=2.3, seed=9)
    c, r = b.ising_create(L, stream=s.cuda_stream, **p), b.ising_create(L, **p)
    try:
        if creutz:
            b.ising_creutz_init(c, None, 3)
        start = b.ising_copy_spins(c, L)
        series = torch.zeros(2 * n, dtype=torch.int64, device="cuda")
        b.ising_sweep_static(c, n, series.data_ptr())
        b.ising_load_spins(c, start, 0)
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=s):
            b.ising_sweep_static(c, n, series.data_ptr())
        b.ising_sweep(r, n)
        _, B, M = b.ising_observables(r, b.ISING_OBS_SERIES)
        for _ in range(3):
            if creutz:
                b.ising_creutz_sweep(c, 2, reverse=True)
            else:
                b.ising_sweep(c, 5)
            b.ising_load_spins(c, start, 0)
            torch.cuda.synchronize()
            graph.replay()
            torch.cuda.synchronize()
            got = series.cpu().numpy()
            assert np.array_equal(got[0::2], B) and np.array_equal(got[1::2], M)
            assert np.array_equal(b.ising_copy_spins(c, L), b.ising_copy_spins(r, L))
    finally:
        b.ising_destroy(c)
        b.ising_destroy(r)


@pytest.mark.parametrize("L", [96, 128, 136, 184])
def test_small_default_sides_are_captured_in_one_workgroup(b, L):
    """ising_sweep and ising_sweep_static of a default context of these sides
    can be captured; every replay equals the eager run."""
    import torch
    G.log(f"captured sweeps of a small default side L={L}")
    s, n = torch.cuda.Stream(), 6
    c, r = b.ising_create(L, h=0.05, T=2.3, seed=L, stream=s.cuda_stream), b.ising_create(L, h=0.05, T=2.3, seed=L)
    try:
        start = b.ising_copy_spins(c, L)
        b.ising_reserve(c, 64)
        series = torch.zeros(2 * n, dtype=torch.int64, device="cuda")
        b.ising_sweep_static(c, n, series.data_ptr())
        b.ising_load_spins(c, start, 0)
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=s):
            b.ising_sweep_static(c, n, series.data_ptr())
            b.ising_sweep(c, n)
        b.ising_sweep(r, 2 * n)
        _, B, M = b.ising_observables(r, b.ISING_OBS_SERIES)
        for _ in range(3):
            b.ising_load_spins(c, start, 0)
            series.fill_(-7)
            torch.cuda.synchronize()
            graph.replay()
            torch.cuda.synchronize()
            got = series.cpu().numpy()
            assert np.array_equal(got[0::2], B[:n]) and np.array_equal(got[1::2], M[:n])
            assert np.array_equal(b.ising_copy_spins(c, L), b.ising_copy_spins(r, L))
        b.ising_plan_set(c, b.ISING_PLAN_BANDS)
        with torch.cuda.graph(torch.cuda.CUDAGraph(), stream=s):
            with pytest.raises(b.IsingError):
                b.ising_sweep(c, 1)
            b.ising_sweep_static(c, 1, series.data_ptr())
    finally:
        b.ising_destroy(c)
        b.ising_destroy(r)


@pytest.mark.parametrize("L,flags,eager,n", [(16392, 0, 20, 16), (16392, 0, 3, 35), (1024, 1, 20, 16), (1024, 1, 3, 35)])
def test_two_pass_sweeps_are_captured_after_eager_ones(b, L, flags, eager, n):
    """Beyond 16384 eager sweeps run over tiles, and those of a two-pass plan
    (flags 1) as replays of a graph of its own; a captured call of any length
    runs as two-pass launches and replays like an eager one."""
    import torch
    G.log(f"captured sweeps of a two-pass side L={L} n={n}")
    s = torch.cuda.Stream()
    c = b.ising_create(L, T=2.3, seed=5, flags=flags, stream=s.cuda_stream)
    r = b.ising_create(L, T=2.3, seed=5, flags=flags)
    try:
        b.ising_reserve(c, 512)
        b.ising_sweep(c, eager)
        start = b.ising_copy_spins(c, L)
        b.ising_load_spins(c, start, 0)
        b.ising_load_spins(r, start, 0)
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=s):
            b.ising_sweep(c, n)
        b.ising_sweep(r, n)
        _, B, M = b.ising_observables(r, b.ISING_OBS_SERIES)
        want = b.ising_copy_spins(r, L)
        for _ in range(3):
            b.ising_load_spins(c, start, 0)
            torch.cuda.synchronize()
            graph.replay()
            torch.cuda.synchronize()
            assert np.array_equal(b.ising_copy_spins(c, L), want)
    finally:
        b.ising_destroy(c)
        b.ising_destroy(r)
