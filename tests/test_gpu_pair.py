"""Two steps in one pass over the lattice (k_pair, k_near) against the same
steps taken one by one: the cell update has every operation written out, so
the two ways agree bit for bit.  Sizes sit at the edges of a block's column
(64 cells along x, 12 rows along z, a few planes along y)."""
import numpy as np
import pytest

import workloads as WL

pytestmark = pytest.mark.gpu

P, W, V, O, ZV, ZO = (WL.PERIODIC, WL.WALL, WL.VELOCITY, WL.PRESSURE, WL.ZH_VELOCITY, WL.ZH_PRESSURE)


def _solve(bx, wings, seed, check_interval=0, step0=0):
    from paper_2102_01305_amd.solver import Solver

    rng = np.random.default_rng(seed)
    shape = (bx["nz"], bx["ny"], bx["nx"])
    u = rng.uniform(-5e-3, 5e-3, (3,) + shape)
    u[0] += (bx.get("u_in") or [0.0])[0]
    s = Solver(bx, wings, check_interval=check_interval, history_steps=64)
    s.init_fields(rho=rng.uniform(0.995, 1.005, shape), u=u, step0=step0)
    return s


def _updates_per_launch(s, run):
    s.enable_timing(1)
    s.read_timing()
    run()
    t = s.read_timing()
    s.enable_timing(0)
    return t["collide_cells"] / t["collide_launches"] / s.N


def _same(a, b, what=("u", "rho", "fdist")):
    for k in what:
        np.testing.assert_array_equal(a.fields(k), b.fields(k), err_msg=k)
    if a.nw:
        n = a.step_count
        np.testing.assert_array_equal(a.forces(n - 12, 12), b.forces(n - 12, 12))
        for k in ("X", "U", "B", "duB", "rhoB"):
            np.testing.assert_array_equal(a.markers(k), b.markers(k), err_msg=k)


@pytest.mark.parametrize("bc", [
    [P] * 6, [V, O, W, W, P, P], [W] * 6, [ZV, ZO, W, W, P, P], [ZO, ZV, P, P, W, W], [P, P, W, W, W, W],
    [W, O, P, P, P, P]], ids=["periodic", "channel", "closed", "zou_he", "zou_he_z_walls", "duct", "wall_out"])
@pytest.mark.parametrize("size,force", [((128, 64, 96), 0.0), ((129, 97, 101), 1e-5), ((65, 127, 133), 0.0)],
                         ids=lambda v: "x".join(map(str, v)) if isinstance(v, tuple) else f"g{v}")
def test_lattice_pairs_equal_single_steps(bc, size, force):
    bx = WL.box(*size, bc, 0.6, u_in=(0.03, 0.002, -0.001) if bc[0] != P else (0, 0, 0), rho_out=1.001,
                body_force=(force, -force, 2 * force))
    print(f"[pair] lattice {size} bc {bc} force {force}", flush=True)
    a, b = _solve(bx, [], 7), _solve(bx, [], 7)
    per = _updates_per_launch(a, lambda: a.step(10))
    assert per == 2.0 if size != (65, 127, 133) else per in (1.0, 2.0)
    a.step(1)                                          # an odd number in all
    for _ in range(11):
        b.step(1)
    _same(a, b)
    a.close()
    b.close()


def test_pairs_step_round_check_steps_and_windows():
    bx = WL.box(128, 64, 96, [P] * 6, 0.6)
    print("[pair] check steps", flush=True)
    a, b = _solve(bx, [], 3, check_interval=5), _solve(bx, [], 3, check_interval=5)
    a.step(71)                                         # past a window of 64 steps
    for _ in range(71):
        b.step(1)
    assert a.mass() == b.mass() and a.mass()[0] == 70
    _same(a, b, ("fdist",))
    a.close()
    b.close()


@pytest.mark.parametrize("case", ["clap_fling", "cylinder", "corner"])
def test_foil_pairs_equal_single_steps(case):
    from paper_2102_01305_amd.solver import complete_case

    if case == "clap_fling":
        bx, wg, ph = WL.clap_fling_case()
    elif case == "cylinder":
        bx, wg, ph = WL.cylinder_case(nx=253, ny=190, nz=187, d=20.0)
    else:
        # periodic all round, the foil's node box at the corner of the box:
        # steps are taken one by one, as its neighbours wrap
        bx, wg, ph = WL.plate_case(nx=256, ny=192, nz=192, centre=(6.2, 6.2))
        bx = dict(bx, bc=[P] * 6, u_in=[0.0, 0.0, 0.0])
    bx, wg = complete_case(bx, wg, ph)
    print(f"[pair] {case}", flush=True)
    a, b = _solve(bx, wg, 11, step0=210), _solve(bx, wg, 11, step0=210)
    assert _updates_per_launch(a, lambda: a.step(12)) == (1.0 if case == "corner" else 2.0)
    for _ in range(12):
        b.step(1)
    _same(a, b, ("u",))
    a.close()
    b.close()


@pytest.mark.parametrize("bc,centre", [([V, O, W, W, P, P], (60.2, 6.4)), ([ZV, ZO, W, W, P, P], (60.2, 184.6)),
                                       ([P] * 6, (245.6, 11.2))], ids=["low_wall", "high_wall", "periodic"])
def test_foil_beside_walls_pairs_equal_single_steps(bc, centre):
    """The cells around a foil that step s is given first (k_near): beside
    a y wall, across the periodic span, near an x face."""
    from paper_2102_01305_amd.solver import complete_case

    bx, wg, ph = WL.plate_case(nx=256, ny=192, nz=192, centre=centre)
    u_in = [0.03, 0.0, 0.0] if bc[0] != P else [0.0, 0.0, 0.0]
    bx, wg = complete_case(dict(bx, bc=bc, u_in=u_in), wg, ph)
    print(f"[pair] plate at {centre} bc {bc}", flush=True)
    a, b = _solve(bx, wg, 5), _solve(bx, wg, 5)
    assert _updates_per_launch(a, lambda: a.step(12)) == 2.0
    for _ in range(12):
        b.step(1)
    _same(a, b, ("u",))
    a.close()
    b.close()


def test_batch_pairs_equal_single_steps():
    from paper_2102_01305_amd.solver import complete_case, step_batch

    print("[pair] batch", flush=True)
    descr = [(WL.box(200, 160, 160, [P] * 6, 0.6), [], 0), (WL.box(130, 61, 97, [V, O, W, W, P, P], 0.6, u_in=(0.02, 0, 0)), [], 0)]
    for nx, ny, nz, c in ((64, 48, 8, 8.0), (97, 80, 81, 10.0), (128, 96, 60, 12.0)):
        bx, wg, ph = WL.clap_fling_case(nx=nx, ny=ny, nz=nz, chord=c)
        descr.append((*complete_case(bx, wg, ph), 40))
    a = [_solve(bx, wg, k, step0=s0) for k, (bx, wg, s0) in enumerate(descr)]
    b = [_solve(bx, wg, k, step0=s0) for k, (bx, wg, s0) in enumerate(descr)]
    step_batch(a, 1)
    step_batch(a, 70)
    for _ in range(71):
        step_batch(b, 1)
    for x, y in zip(a, b):
        _same(x, y, ("u", "fdist"))
        x.close()
        y.close()
