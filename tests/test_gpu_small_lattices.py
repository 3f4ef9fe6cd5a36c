"""GPU parity of the smallest resident lattices (a thread keeps one, two or
four words of each colour in registers) against the oracle: sides from one
word a row to the largest, around the limits of a word per thread, alone (the
resident plan, a workgroup of as many waves as the lattice has words for) and
in a resident batch (1024 threads), fields, J < 0, zero thresholds, certain
flips, and runs across the flush of the per-sweep sums."""
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


RUNS = [W.Run(L=8, T=2.0, seed=1, sweeps=70), W.Run(L=16, h=0.1, T=2.3, seed=2, sweeps=129), W.Run(L=24, J=-1.0, T=1.7, seed=3, sweeps=9),
        W.Run(L=64, T=2.27, seed=4, sweeps=65), W.Run(L=72, h=-0.4, T=0.2, seed=5, sweeps=12), W.Run(L=88, T=1e300, seed=6, sweeps=3),
        W.Run(L=96, h=0.05, T=2.27, seed=7, sweeps=11), W.Run(L=128, T=2.27, seed=8, sweeps=64, p_up=1.0),
        W.Run(L=136, J=0.5, h=0.2, T=1.1, seed=9, sweeps=10), W.Run(L=176, T=2.27, seed=10, sweeps=7), W.Run(L=184, h=0.1, T=2.0, seed=11, sweeps=6)]


def _check(b, o, run, ctx, what):
    obs, B, M = b.ising_observables(ctx, b.ISING_OBS_SERIES | b.ISING_OBS_HASH)
    got = {"spins": b.ising_copy_spins(ctx, run.L), "B": B, "M": M, "hash": obs.lattice_hash}
    G.assert_same(got, G.oracle_run(o, run), what)


@pytest.mark.parametrize("run", RUNS, ids=lambda r: f"L{r.L}")
def test_resident_plan(b, o, run):
    G.log(f"small lattice alone {run}")
    ctx = b.ising_create(run.L, run.J, run.h, run.T, run.seed, run.p_up)
    try:
        b.ising_plan_set(ctx, b.ISING_PLAN_RESIDENT)
        for n in (1, run.sweeps - 1):
            b.ising_sweep(ctx, n)
        _check(b, o, run, ctx, f"L={run.L}")
    finally:
        b.ising_destroy(ctx)


def test_resident_batch(b, o):
    ctxs = [b.ising_create(r.L, r.J, r.h, r.T, r.seed, r.p_up) for r in RUNS]
    try:
        G.log("small lattices, one resident batch")
        b.ising_sweep_batch_plan(ctxs, [r.sweeps for r in RUNS], b.ISING_BATCH_RESIDENT)
        for r, c in zip(RUNS, ctxs):
            _check(b, o, r, c, f"batch L={r.L}")
    finally:
        for c in ctxs:
            b.ising_destroy(c)
