"""Which kernels a call goes to, on the host side alone: the library's HIP
calls are served by host memory, its launches counted."""
import pytest

from tests import hip_host


@pytest.mark.parametrize("L,h", [(4104, 0.1), (16392, 0.0)])
def test_a_forced_plan_runs_as_it_is(L, h):
    """Beyond the row bands AUTO sweeps between two buffers (wave tiles); a
    plan that the caller forces, at creation or later, runs in its own."""
    hip_host.run(f"""
        L = {L}
        plan = b.ISING_PLAN_BANDS if L <= 16384 else b.ISING_PLAN_TWO_PASS
        def sweep(c):
            b.ising_reserve(c, 1024)
            b.ising_sweep(c, 1)
            n, live = h.cooperative, h.live
            b.ising_sweep(c, 3)
            return h.cooperative - n, h.live - live >= L * L
        banded = 1 if L <= 16384 else 0
        auto = b.ising_create(L, h={h})
        assert b.ising_plan_info(auto)[0] == plan
        assert sweep(auto) == (0, True)
        assert sweep(b.ising_create(L, h={h}, flags=plan)) == (banded, False)
        c = b.ising_create(L, h={h})
        b.ising_plan_set(c, plan)
        assert sweep(c) == (banded, False)
    """)


@pytest.mark.parametrize("trial", [4, 20])
def test_a_tuned_default_runs_as_before(trial):
    """The plan of the side, when nothing beats it, goes on being run with its
    wave tiles, on the tuned context and on later ones."""
    hip_host.run(f"""
        c = b.ising_create(4104, h=0.1)
        info = b.ising_plan_info(c)
        b.ising_tune(c, {trial})
        assert b.ising_plan_info(c) == info
        for ctx in (c, b.ising_create(4104, h=0.1)):
            n = h.cooperative
            b.ising_sweep(ctx, 3)
            assert h.cooperative == n
    """)


@pytest.mark.parametrize("L", [96, 136, 184])
def test_a_tuned_default_is_captured_as_before(L):
    """ising_sweep of these sides can be captured; tuning that keeps the plan
    changes nothing."""
    hip_host.run(f"""
        c = b.ising_create({L})
        b.ising_tune(c, 4)
        for ctx in (c, b.ising_create({L})):
            b.ising_reserve(ctx, 8)
            h.capturing = 1
            b.ising_sweep(ctx, 3)
            h.capturing = 0
    """)


@pytest.mark.parametrize("L", [136, 184])
def test_short_calls_of_a_forced_band_plan_run_on_bands(L):
    """Only AUTO's choice gives short calls of small sides to one workgroup;
    ising_tune's band shapes are each timed on the band kernel."""
    hip_host.run(f"""
        def launches(c, n):
            k = h.cooperative
            b.ising_sweep(c, n)
            return h.cooperative - k
        auto, forced = b.ising_create({L}), b.ising_create({L}, flags=b.ISING_PLAN_BANDS)
        assert launches(auto, 1) == 0 and launches(auto, 2) == 0 and launches(auto, 30) == 1
        assert launches(forced, 1) == 1 and launches(forced, 2) == 1
        b.ising_plan_set(auto, b.ISING_PLAN_BANDS, 1, 8)
        assert launches(auto, 1) == 1
        k = h.cooperative
        b.ising_tune(b.ising_create({L}), 2)
        # heights 4 (the default: AUTO's), 2, 8, 16 and 32, three rounds, a warm-up of one sweep each
        assert h.cooperative - k == 3 * 4 * 2, h.cooperative - k
    """)


@pytest.mark.parametrize("L", [96, 104, 128])
def test_small_lattices_of_several_streams_share_the_chip(L):
    """Sweeps of default contexts of these sides are single workgroups, which
    run side by side on several streams; band launches are cooperative, one
    at a time."""
    hip_host.run(f"""
        for c in [b.ising_create({L}) for _ in range(4)]:
            for n in (1, 20, 600):
                b.ising_sweep(c, n)
        assert h.cooperative == 0 and h.launches >= 12
    """)


@pytest.mark.parametrize("L", [4096, 6000])
def test_read_backs_into_pinned_memory_are_one_copy(L):
    """A large lattice or its demons go straight into pinned memory, and
    through the ring of chunks into any other."""
    hip_host.run(f"""
        N = {L} * {L}
        c = b.ising_create({L})
        b.ising_creutz_init(c, None, 1)
        pinned, pageable = ctypes.c_void_p(), np.empty(N, dtype=np.int8)
        assert lib.hipHostMalloc(ctypes.byref(pinned), ctypes.c_size_t(N), 0) == 0
        for read in (b.lib().ising_copy_spins, b.lib().ising_copy_demons):
            for dst, copies in ((pinned.value, 1), (pageable.ctypes.data, -(-N // (2 << 20)))):
                n = h.copies
                assert read(c, dst, N) == 0
                assert h.copies - n == copies, (h.copies - n, copies)
    """)


@pytest.mark.parametrize("L,direct", [(66, True), (258, True), (398, True), (402, False), (1002, False)])
def test_single_sweeps_of_small_partial_word_sides(L, direct):
    """One sweep of such a side is faster as per-site launches up to 400."""
    hip_host.run(f"""
        c = b.ising_create({L})
        b.ising_sweep(c, 1)
        assert h.cooperative == {0 if direct else 1}
        b.ising_sweep(c, 2)
        assert h.cooperative == {1 if direct else 2}
    """)


@pytest.mark.parametrize("L", [96, 184, 1024])
def test_a_lone_batch_on_a_captured_stream_is_refused(L):
    """Its band launches cannot be replayed: the edge words of one replay
    carry the tags that the next one waits for."""
    hip_host.run(f"""
        c = b.ising_create({L})
        b.ising_sweep_batch([c], [3])
        assert h.cooperative == 1
        h.capturing = 1
        for stream in (None, 1):
            try:
                b.ising_sweep_batch([c], [3], stream=stream)
            except b.IsingError as e:
                assert e.code == b.ISING_EUNSUPPORTED
            else:
                raise AssertionError("captured")
        h.capturing = 0
        b.ising_sweep_batch([c], [3])
        assert h.cooperative == 2 and b.ising_observables(c)[0].sweeps_done == 6
    """)
