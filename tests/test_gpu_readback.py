"""Whole lattices, demon maps and arrival maps read back to ordinary host
memory: sides around the size from which the copy goes through pinned chunks
(16 MiB), a last chunk that is not whole, sides of each word layout (whole
groups of four words a row, single words, partial words), buffers of torch at
a site's alignment, several threads at once, and the way back in."""
import threading

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


@pytest.mark.parametrize("L", [2, 8, 24, 30, 96, 1000, 1026, 4088, 4096, 4098, 4104, 5800])
def test_spins_and_demons_round_trip(b, L):
    s, d = W.random_lattice(L, L), W.random_demons(L, L + 1, 255)
    G.log(f"round trip L={L}")
    c = b.ising_create(L)
    try:
        b.ising_load_spins(c, s, 3)
        assert np.array_equal(b.ising_copy_spins(c, L), s)
        b.ising_creutz_init(c, d)
        assert np.array_equal(b.ising_copy_demons(c, L), d)
        assert np.array_equal(b.ising_copy_spins(c, L), s)
    finally:
        b.ising_destroy(c)


@pytest.mark.parametrize("L,offset", [(104, 4), (64, 8), (102, 1), (256, 4)])
def test_caller_buffers_of_any_alignment(b, L, offset):
    """A caller's buffer aligned to 4 or 8 bytes (whole words), or to one
    byte where a row does not hold whole words."""
    import torch
    n = b.ising_state_bytes(L, b.ISING_PLAN_AUTO if L % 8 else b.ISING_PLAN_BANDS)
    buf = torch.zeros(n + 64, dtype=torch.uint8, device="cuda")
    s = W.random_lattice(L, 5)
    G.log(f"caller's buffer L={L} offset={offset}")
    c = b.ising_create_in(buf.data_ptr() + offset, n, L, flags=b.ISING_PLAN_AUTO if L % 8 else b.ISING_PLAN_BANDS)
    try:
        b.ising_load_spins(c, s, 0)
        assert np.array_equal(b.ising_copy_spins(c, L), s)
    finally:
        b.ising_destroy(c)
    assert not buf[:offset].any() and not buf[offset + n:].any()


@pytest.mark.parametrize("L,n", [(2, 1), (64, 4096), (254, 4097), (256, 4096), (258, 4097), (264, 40)])
def test_small_read_backs(b, L, n):
    """Sides and series lengths around the sizes up to which a kernel writes
    the read-back into host memory (256^2 sites, 4096 sweeps) and one call
    brings the series: the whole series, the hash and the spins
    equal those of twin runs read back in other ways, also with a prefetched
    read-back in the stage, which stays good."""
    from oracle import ref
    o = ref.default()
    want = b.ISING_OBS_SERIES | b.ISING_OBS_HASH
    G.log(f"small read-back L={L} n={n}")
    one, two = b.ising_create(L, seed=5), b.ising_create(L, seed=5)
    try:
        b.ising_sweep(one, n)
        b.ising_sweep(two, n)
        assert b.ising_prefetch_observables(two, want)
        spins = b.ising_copy_spins(two, L)
        obs, B, M = b.ising_observables(one, want)
        obs2, B2, M2 = b.ising_observables(two, want, capacity=n)
        assert len(B) == n and np.array_equal(B, B2) and np.array_equal(M, M2)
        assert np.array_equal(b.ising_copy_spins(one, L), spins)
        assert obs.lattice_hash == obs2.lattice_hash == o.fnv1a64(spins)
        assert (obs.bond_sum, obs.mag_sum) == (B[-1], M[-1]) and M[-1] == spins.sum(dtype=np.int64)
        assert b.ising_observables(one, b.ISING_OBS_SERIES)[0].series_len == 0
    finally:
        b.ising_destroy(one)
        b.ising_destroy(two)


def test_several_threads_read_back_at_once(b):
    """More readers than stages, each on its own context: every lattice
    arrives whole."""
    sides = [4096, 4104, 5000, 4400]
    lattices = [W.random_lattice(L, 70 + L) for L in sides]
    ctxs = [b.ising_create(L) for L in sides]
    try:
        for c, s in zip(ctxs, lattices):
            b.ising_load_spins(c, s, 0)
        G.log("four threads read back")
        got = [None] * len(sides)

        def read(k):
            for _ in range(3):
                got[k] = b.ising_copy_spins(ctxs[k], sides[k])

        threads = [threading.Thread(target=read, args=(k,)) for k in range(len(sides))]
        for t in threads:
            t.start()
        for t in threads:
            t.join()
        for g, s in zip(got, lattices):
            assert np.array_equal(g, s)
    finally:
        for c in ctxs:
            b.ising_destroy(c)


def test_arrival_map_in_chunks(b):
    """A 2060^2 arrival map (16.97 MB: nine chunks, the last not whole)
    equals its pieces' sum and the medium's solid sites."""
    L = 2060
    c = b.perc_create(L, 0.7, 3)
    try:
        b.perc_run(c)
        G.log("arrival map 2060")
        pore, arr, r = b.perc_copy_medium(c, L), b.perc_copy_arrival(c, L), b.perc_result_get(c)
    finally:
        b.perc_destroy(c)
    assert (arr[pore == 0] == -1).all()
    assert (arr >= 0).sum() == r.invaded and arr.max() == r.passes and pore.sum(dtype=np.int64) == r.pores
