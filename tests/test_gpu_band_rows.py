"""GPU parity of the band kernel that keeps a wave per row against the
oracle: rows that fill a wave's words, that end inside a wave (the word
after the last is a copy of the first) and that start inside a word (sides
that are not multiples of 8), one to eight words a lane, bands of one row
to sixteen, uneven bands, each number of half-sweeps between exchanges,
calls that end inside a block of them and that cross the flush and launch
limits, and the short calls that other kernels serve."""
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


def _run(b, run, rows, calls):
    ctx = b.ising_create(run.L, run.J, run.h, run.T, run.seed, run.p_up)
    try:
        if rows:
            b.ising_plan_set(ctx, b.ISING_PLAN_BANDS, 1, rows)
        for n in calls:
            b.ising_sweep(ctx, n)
        obs, B, M = b.ising_observables(ctx, b.ISING_OBS_SERIES | b.ISING_OBS_HASH)
        return {"spins": b.ising_copy_spins(ctx, run.L), "B": B, "M": M, "hash": obs.lattice_hash}
    finally:
        b.ising_destroy(ctx)


# L, J, h, T, band rows (0: the default), calls
CASES = [
    # rows that fill a wave: 1, 2, 3, 4, 5, 6, 7 and 8 words a lane
    (512, 1.0, 0.0, 2.27, 4, [7, 1, 2, 35]),
    (512, 1.0, 0.05, 2.0, 2, [5, 3]),
    (1024, -1.0, 0.1, 1.5, 4, [3, 70]),
    (1536, 1.0, 0.0, 2.27, 6, [5]),
    (2048, 1.0, 0.0, 0.2, 8, [1, 3]),      # zero thresholds
    (2560, 1.0, 0.0, 2.27, 10, [3]),
    (3072, 1.0, 0.05, 2.27, 12, [3]),
    (3584, 1.0, 0.0, 1e300, 14, [2]),      # every proposal accepted
    (4096, 1.0, 0.0, 2.27, 16, [3]),
    # rows that end inside a wave, uneven bands
    (72, 1.0, 0.0, 2.27, 1, [9]),
    (200, 1.0, 0.3, 2.0, 7, [9]),
    (520, 1.0, 0.0, 2.27, 3, [6, 3]),      # 65 words: two a lane, the second lane's ghost
    (1000, 1.0, 0.0, 2.27, 4, [9]),
    (1528, 0.5, -0.2, 2.5, 5, [4]),
    (2056, 1.0, 0.1, 2.27, 9, [3]),
    (3080, 1.0, 0.1, 2.27, 13, [3]),
    (4088, 1.0, 0.0, 2.27, 16, [2]),
    # rows that start inside a word (L % 8 = 2, 4, 6)
    (4, 1.0, 0.0, 2.27, 0, [5]),
    (10, 1.0, 0.1, 2.27, 0, [5, 4]),
    (18, 1.0, 0.0, 2.27, 0, [1, 9]),
    (34, -1.0, 0.2, 2.0, 0, [3]),
    (102, 1.0, 0.0, 2.27, 0, [41]),
    (252, 1.0, 0.1, 0.3, 0, [9]),
    (508, 1.0, 0.0, 2.27, 0, [4]),         # the last ghost in the wave's last word
    (510, 1.0, 0.0, 2.27, 0, [4]),         # two words a lane
    (1002, 1.0, 0.0, 2.27, 0, [7, 2]),
    (1366, 1.0, 0.1, 2.27, 0, [4]),
    (2042, 1.0, 0.0, 2.27, 0, [3]),
    (2554, 1.0, 0.0, 2.27, 0, [3]),
    (3062, 1.0, 0.1, 2.27, 0, [3]),
    (4086, 1.0, 0.0, 2.27, 0, [2]),
    (4094, 1.0, 0.0, 2.27, 0, [2]),        # 513 words: the per-site kernels
]


@pytest.mark.parametrize("L,J,h,T,rows,calls", CASES)
def test_band_rows_equal_oracle(b, o, L, J, h, T, rows, calls):
    run = W.Run(L=L, J=J, h=h, T=T, seed=1000 + L, p_up=0.5, sweeps=sum(calls))
    G.log(f"band rows L={L} rows={rows} J={J} h={h} T={T} calls={calls}")
    G.assert_same(_run(b, run, rows, calls), G.oracle_run(o, run), f"L={L} rows={rows}")


@pytest.mark.parametrize("L", [64, 96, 128, 136, 184, 66, 250])
def test_calls_of_every_length_equal_oracle(b, o, L):
    """Small lattices take short and long calls on different kernels; the
    launch limit of 512 sweeps is crossed."""
    calls = [1, 2, 3, 8, 30, 1, 520, 2]
    run = W.Run(L=L, h=0.02, T=2.3, seed=7, sweeps=sum(calls))
    G.log(f"calls of every length L={L}")
    G.assert_same(_run(b, run, 0, calls), G.oracle_run(o, run), f"L={L}")


def test_odd_side_static_and_captured(b):
    """A side that is not a multiple of 8 through ising_sweep_static, eager
    (bands) and captured into a graph (per-site launches), replayed: equal to
    ising_sweep each time."""
    import torch
    L, n = 102, 6
    s = torch.cuda.Stream()
    ref = b.ising_create(L, 1.0, 0.05, 2.3, 41, 0.5)
    ctx = b.ising_create(L, 1.0, 0.05, 2.3, 41, 0.5, stream=s.cuda_stream)
    try:
        start = b.ising_copy_spins(ctx, L)
        b.ising_sweep(ref, n)
        _, B, M = b.ising_observables(ref, b.ISING_OBS_SERIES)
        want = b.ising_copy_spins(ref, L)
        series = torch.full((2 * n,), -7, dtype=torch.int64, device="cuda")
        torch.cuda.synchronize()
        G.log("static sweeps, eager")
        b.ising_sweep_static(ctx, n, series.data_ptr())
        assert np.array_equal(b.ising_copy_spins(ctx, L), want)
        assert np.array_equal(series.cpu().numpy().reshape(n, 2), np.stack([B, M], 1))
        b.ising_load_spins(ctx, start, 0)
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=s):
            b.ising_sweep_static(ctx, n, series.data_ptr())
        for rep in range(3):
            G.log(f"static sweeps, replay {rep}")
            b.ising_load_spins(ctx, start, 0)
            series.fill_(-7)
            torch.cuda.synchronize()
            graph.replay()
            torch.cuda.synchronize()
            assert np.array_equal(series.cpu().numpy().reshape(n, 2), np.stack([B, M], 1)), rep
            assert np.array_equal(b.ising_copy_spins(ctx, L), want), rep
        del graph
    finally:
        b.ising_destroy(ctx)
        b.ising_destroy(ref)
