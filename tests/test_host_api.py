"""The host side of the C ABI on a CPU (host_runtime.cpp stands in for the HIP
runtime and the kernels): which stream, thread and device its work is put on,
and what a call leaves behind."""
import ctypes as C
import threading

import numpy as np
import pytest

import host_runtime as H
import workloads as WL
from paper_2102_01305_amd import _lib as L

P = WL.PERIODIC
W = np.array([1 / 3] + [1 / 18] * 6 + [1 / 36] * 12)[:, None, None, None]


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    return H.build(tmp_path_factory.mktemp("host_side"))


def _transfers(s):
    """Fields of a few chunks up and down, checked value by value."""
    n = int(np.prod(s.shape))
    f = W + np.random.default_rng(n).uniform(-2e-2, 2e-2, (19,) + s.shape)
    s.init(fdist=f)
    np.testing.assert_array_equal(s.fields(L.FIELD_FDIST), W + (f - W).astype(np.float32).astype(np.float64))
    want = (np.arange(4 * n) % 65521).astype(np.float64)
    np.testing.assert_array_equal(s.fields(L.FIELD_RHO).reshape(-1), want[:n])
    np.testing.assert_array_equal(s.fields(L.FIELD_U).reshape(-1), want[n:])


@pytest.mark.parametrize("stream", ["null", "own", "per_thread"])
def test_transfers_come_after_the_kernels_of_any_kind_of_stream(lib, stream):
    st = {"null": None, "own": lib.host_stream(0), "per_thread": H.PER_THREAD}[stream]
    s = H.Solve(lib, WL.box(130, 70, 69, [P] * 6, 0.6), stream=st)   # 2.4 MB a population: 23 chunks
    _transfers(s)
    s.close()


def test_transfers_with_another_device_current(lib):
    """A solve made on one device is read and written with another current,
    and the current device stays what it was."""
    lib.host_device(1)
    s = H.Solve(lib, WL.box(130, 70, 69, [P] * 6, 0.6), stream=lib.host_stream(1))
    for current in (0, 1, 0):
        lib.host_device(current)
        _transfers(s)
        assert lib.host_current() == current
    # and on a stream of the other device from then on
    s.check(lib.ibmlbm_set_stream(s.h, C.c_void_p(lib.host_stream(0))))
    lib.host_device(1)
    _transfers(s)
    lib.host_device(0)
    s.close()


def test_pinned_staging_is_bounded_for_all_solves_and_given_back(lib):
    assert lib.host_pinned(0) == 0
    made = [H.Solve(lib, WL.box(130, 70, 69, [P] * 6, 0.6), stream=lib.host_stream(0)) for _ in range(8)]
    handles = lib.host_pinned(0)                       # what each handle holds for its launch arguments
    for s in made:
        _transfers(s)
    assert lib.host_pinned(0) - handles <= 64 << 20
    errors = []

    def go(s):
        try:
            _transfers(s)
        except AssertionError as e:
            errors.append(e)

    threads = [threading.Thread(target=go, args=(s,)) for s in made]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not errors
    assert lib.host_pinned(1) - handles <= 64 << 20    # however many at once
    for s in made:
        s.close()
    assert lib.host_pinned(0) == 0
    one = H.Solve(lib, WL.box(130, 70, 69, [P] * 6, 0.6))
    handles = lib.host_pinned(0)
    _transfers(one)
    _transfers(one)
    assert lib.host_pinned(0) - handles <= 16 << 20    # a single solve: the staging of one transfer
    one.close()
    assert lib.host_pinned(0) == 0


@pytest.mark.parametrize("slots", [0, 1, 3])
def test_transfers_without_pinned_memory_left(lib, slots):
    solves = [H.Solve(lib, WL.box(130, 70, 69, [P] * 6, 0.6), stream=lib.host_stream(0)) for _ in range(2)]
    lib.host_fail(b"pinned", slots)
    for s in solves + solves:
        _transfers(s)
    lib.host_fail(b"", 0)
    for s in solves:
        s.close()
    assert lib.host_pinned(0) == 0


@pytest.mark.parametrize("size,copied", [((4, 4, 1), False), ((27, 73, 7), False), ((69, 200, 1), True)],
                         ids=lambda v: "x".join(map(str, v)) if isinstance(v, tuple) else None)
def test_small_transfers_make_no_copy(lib, size, copied):
    """Up to 1 MB (13797 cells for the populations) the kernel itself reads or
    writes the pinned slot."""
    s = H.Solve(lib, WL.box(*size, [P] * 6, 0.6), stream=H.PER_THREAD)
    before = lib.host_copies()
    _transfers(s)
    assert (lib.host_copies() > before) == copied
    s.close()


def _foil_solve(lib, nx=256, ny=192, nz=192, chord=20.0, step0=0, **kw):
    import oracle.params as params

    bx, wg, ph = WL.clap_fling_case(nx=nx, ny=ny, nz=nz, chord=chord)
    bx, wg = params.complete_case(bx, wg, ph)
    s = H.Solve(lib, bx, wg, **kw)
    s.init(step0=step0)
    return s


def _steps_done(s):
    """Steps that the solve's current state has seen: the further of the two
    states (the idle one is older, or was written by a step not yet taken)."""
    s.check(s.lib.ibmlbm_mass(s.h, C.byref(C.c_int64()), C.byref(C.c_double())))   # (waits for the stream)
    return max(int(v[0]) for v in s.state)


@pytest.mark.parametrize("kind,after", [("factor", 0), ("markers", 0), ("near", 0), ("markers", 1), ("pair", 0),
                                        ("markers", 3), ("pair", 1)])
def test_an_error_between_the_steps_of_a_pair_loses_no_step(lib, kind, after):
    """The step count stays that of the state the solve still has, and the
    next call goes on from there."""
    s = _foil_solve(lib)
    lib.host_calls()
    lib.host_fail(kind.encode(), after)
    assert lib.ibmlbm_step(s.h, 10) == L.EDEVICE
    assert s.step_count() == _steps_done(s)
    lib.host_calls()
    s.check(lib.ibmlbm_step(s.h, 70 - s.step_count()))
    calls = lib.host_calls().decode().split()
    assert calls[0] == "factor" and "pair" in calls    # (the failed window is made again)
    assert s.step_count() == _steps_done(s) == 70
    s.close()


def _launches(lib, run):
    lib.host_calls()
    run()
    return lib.host_calls().decode().splitlines()


def test_solves_of_the_pair_tests_are_planned_in_pairs(lib):
    """What test_gpu_pair_paths.py compares with single steps does take pairs:
    alone, and in a batch with first, second and single steps side by side."""
    import oracle.params as params
    import pair_cases as PC

    solves = [(PC.lattice(size, bc), []) for size in PC.RAGGED for bc in PC.FACES.values()]
    solves += [PC.foil(c, params.complete_case) for c in ("clap_fling", "cylinder", "plate")]
    for bx, wg in solves:
        s = H.Solve(lib, bx, wg)
        s.init()
        calls = _launches(lib, lambda: s.check(lib.ibmlbm_step(s.h, 12)))
        assert calls.count("pair 1") == 6 and "collide 1" not in calls, bx
        s.close()

    made = []
    for bx, wg, storage, check, step0, alone in PC.batch(params.complete_case):
        made.append(H.Solve(lib, bx, wg, storage=storage, check_interval=check))
        made[-1].init(step0=step0)
        made[-1].check(lib.ibmlbm_step(made[-1].h, alone))
    group = (L.Handle * len(made))(*[s.h for s in made])
    calls = _launches(lib, lambda: made[0].check(lib.ibmlbm_step_batch(group, len(made), 70)))
    count = {k: [int(c.split()[1]) for c in calls if c.startswith(k)] for k in ("near", "pair", "collide")}
    assert max(count["near"]) >= 4 and max(count["pair"]) >= 4 and max(count["collide"]) >= 2
    alt = [(int(c.split()[1]), int(c.split()[3])) for c in calls if c.startswith("markers")]
    assert len({m for n, m in alt if n >= 4 and 0 < m < (1 << n) - 1}) >= 4   # groups with both kinds of source
    for s, (_, _, _, _, step0, alone) in zip(made, PC.batch(params.complete_case)):
        assert s.step_count() - step0 == _steps_done(s) == 70 + alone
        s.close()
