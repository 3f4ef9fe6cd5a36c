"""The library's host side under failures that a GPU run cannot ask for, with
its HIP calls served by host memory."""
import pytest

from tests import hip_host


@pytest.mark.parametrize("L,plan", [(2048, "AUTO"), (96, "BANDS"), (1002, "AUTO")])
def test_band_memory_stays_when_it_cannot_grow(L, plan):
    """Creutz bands take more edge words than Metropolis bands. Where those
    are not to be had the sweeps run without bands (or, where that takes a
    second lattice, are refused), and the words and partial sums that the band
    plan has are still there for its next launch."""
    hip_host.run(f"""
        c = b.ising_create({L}, flags=b.ISING_PLAN_{plan})
        b.ising_creutz_init(c, None, 1)
        b.ising_reserve(c, 64)
        b.ising_sweep(c, 40)
        assert h.cooperative == 1
        live = h.live
        h.fail_malloc = 0
        try:
            b.ising_creutz_sweep(c, 5)
        except b.IsingError as e:
            assert e.code == b.ISING_ENOMEM and {L} % 512 == 0
        assert h.cooperative == 1 and h.live == live, (h.cooperative, live, h.live)
        b.ising_sweep(c, 20)
        assert h.cooperative == 2
        h.fail_malloc = -1
        b.ising_creutz_sweep(c, 5)
        assert h.cooperative == 3 and h.live > live
    """)


@pytest.mark.parametrize("read", ["ising_copy_demons(c, 1024)", "ising_demon_sum(c)", "ising_copy_spins(c, 1024)",
                                  "ising_observables(c)"])
def test_an_edge_wait_that_gave_up_is_reported(read):
    """A band launch of Creutz sweeps that marks a time-out leaves no valid
    state: every read-back says so."""
    hip_host.run(f"""
        c = b.ising_create(1024)
        b.ising_creutz_init(c, None, 1)
        b.ising_creutz_sweep(c, 5)
        b.{read}
        h.mark = 1
        b.ising_creutz_sweep(c, 5)
        assert h.cooperative == 2
        try:
            b.{read}
        except b.IsingError as e:
            assert e.code == b.ISING_EDEVICE, e.code
        else:
            raise AssertionError("no error")
    """)


@pytest.mark.parametrize("fail,cpus", [("new", 8), ("set_device", 8), ("set_device", 1)])
def test_large_read_backs_go_on_without_helpers(fail, cpus):
    """A copy helper that cannot be started, or cannot set its device, is done
    without: the calling thread moves what is left, every byte of it."""
    hip_host.run(f"""
        import os
        os.sched_setaffinity(0, sorted(os.sched_getaffinity(0))[:{cpus}])
        L = 6000
        c = b.ising_create(L)
        for k in range(3):
            out = np.full((L, L), 7, dtype=np.int8)
            h.fail_{fail} = 1 if k else -1  # the first copy allocates the ring
            rc = b.lib().ising_copy_spins(c, out.ctypes.data, out.size)
            h.fail_{fail} = -1
            assert rc == 0 and not out.any(), rc
    """)


def test_a_per_site_context_needs_no_room_for_bands():
    """Sides that are not multiples of 8 run on bands where there is memory
    for their words and partial sums; without it the context is created all
    the same and runs per-site launches."""
    hip_host.run("""
        for k in range(8):
            h.fail_malloc = k  # the lattice, the observables' scratch, then the bands' memory
            try:
                c = b.ising_create(1002)
            except b.IsingError as e:
                assert e.code == b.ISING_ENOMEM and k < 2, (k, e.code)
                continue
            finally:
                h.fail_malloc = -1
            n, m = h.cooperative, h.launches
            b.ising_sweep(c, 3)
            assert h.cooperative - n == (1 if k >= 4 else 0), (k, h.cooperative - n)
            assert k >= 4 or h.launches - m >= 9
            b.ising_copy_spins(c, 1002)
            b.ising_destroy(c)
    """)
