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


@pytest.mark.parametrize("L,hi,calls", [(4104, 255, [4, -5]), (5000, 4, [-4, 6]), (8192, 3, [4, -4]), (8200, 255, [7]),
                                        (10000, 3, [-4, 4]), (16384, 3, [4]), (16392, 3, [-4]), (20016, 4, [4])])
def test_calls_of_several_pairs_equal_oracle(b, o, L, hi, calls):
    """One to three launches of two sweeps, zero to three single sweeps."""
    test_creutz_pairs_equal_oracle(b, o, L, hi, calls)


@pytest.mark.parametrize("L,captured,eager", [(4104, "reverse", [-2]), (4104, "reverse", [3, -7]), (4104, "static", [6]),
                                              (8192, "static", [2]), (8192, "static", [6, -2]), (8192, "reverse", [-6])])
def test_captured_graphs_stay_valid(b, L, captured, eager):
    """A graph of reversed Creutz sweeps or of static Metropolis sweeps holds
    the addresses of the lattice and the demons: after eager Creutz calls a
    replay goes on from where they ended."""
    import torch
    G.log(f"graph of {captured} sweeps after eager Creutz calls L={L} eager={eager}")
    s, p = torch.cuda.Stream(), dict(J=1.0, h=0.0, T=2.3, seed=9)
    c, r = b.ising_create(L, stream=s.cuda_stream, **p), b.ising_create(L, **p)
    demons = W.random_demons(L, 5, 3)
    try:
        for ctx in (c, r):
            b.ising_reserve(ctx, 256)
        series = torch.zeros(4, dtype=torch.int64, device="cuda")
        spins = b.ising_copy_spins(c, L)

        def sweep(ctx):
            if captured == "static":
                b.ising_sweep_static(ctx, 2, series.data_ptr())
            else:
                b.ising_creutz_sweep(ctx, 2, reverse=True)

        def restart(ctx):
            b.ising_load_spins(ctx, spins, 0)
            b.ising_creutz_init(ctx, demons)

        b.ising_creutz_init(c, demons)
        for n in (8, -8):  # every buffer that eager calls take is there
            b.ising_creutz_sweep(c, abs(n), n < 0)
        sweep(c)
        restart(c)
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=s):
            sweep(c)
        for _ in range(3):
            restart(c)
            restart(r)
            for ctx in (c, r):
                for n in eager:
                    b.ising_creutz_sweep(ctx, abs(n), n < 0)
            torch.cuda.synchronize()
            graph.replay()
            torch.cuda.synchronize()
            sweep(r)
            torch.cuda.synchronize()
            assert np.array_equal(b.ising_copy_spins(c, L), b.ising_copy_spins(r, L))
            assert np.array_equal(b.ising_copy_demons(c, L), b.ising_copy_demons(r, L))
    finally:
        b.ising_destroy(c)
        b.ising_destroy(r)


@pytest.mark.parametrize("L,eager", [(512, [40]), (1024, [5, -5]), (8192, [4])])
def test_forward_sweeps_are_captured_after_eager_ones(b, L, eager):
    """Sides with wave tiles, whose eager calls run on bands or by pairs: a
    forward call is captured without allocating, and replays like an eager
    one."""
    import torch
    G.log(f"captured forward Creutz sweeps L={L}")
    s, n, p = torch.cuda.Stream(), 2, dict(J=1.0, h=0.0, T=2.3, seed=9)
    c, r = b.ising_create(L, stream=s.cuda_stream, **p), b.ising_create(L, **p)
    demons = W.random_demons(L, 5, 3)
    try:
        spins = b.ising_copy_spins(c, L)
        for ctx in (c, r):
            b.ising_creutz_init(ctx, demons)
            b.ising_reserve(ctx, 256)
            for k in eager:
                b.ising_creutz_sweep(ctx, abs(k), k < 0)
            b.ising_load_spins(ctx, spins, 0)
            b.ising_creutz_init(ctx, demons)
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=s):
            b.ising_creutz_sweep(c, n)
        b.ising_creutz_sweep(r, n)
        for _ in range(3):
            b.ising_load_spins(c, spins, 0)
            b.ising_creutz_init(c, demons)
            torch.cuda.synchronize()
            graph.replay()
            torch.cuda.synchronize()
            assert np.array_equal(b.ising_copy_spins(c, L), b.ising_copy_spins(r, L))
            assert np.array_equal(b.ising_copy_demons(c, L), b.ising_copy_demons(r, L))
    finally:
        b.ising_destroy(c)
        b.ising_destroy(r)
