"""Two steps in one pass against the same steps one by one, bit for bit, where
a block's column is ragged and on the paths that only some solves take: a last
column of one cell, a last tile of one row, foils with a body force, and groups
with first, second and single steps side by side.  test_host_api.py checks on
the CPU that these solves are planned in pairs."""
import numpy as np
import pytest

import pair_cases as PC
from test_gpu_pair import _same, _solve, _updates_per_launch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("bc", list(PC.FACES.values()), ids=list(PC.FACES))
@pytest.mark.parametrize("size", PC.RAGGED, ids=lambda v: "x".join(map(str, v)))
def test_ragged_lattice_pairs_equal_single_steps(size, bc):
    print(f"[pair] lattice {size} bc {bc}", flush=True)
    bx = PC.lattice(size, bc)
    a, b = _solve(bx, [], 7), _solve(bx, [], 7)
    assert _updates_per_launch(a, lambda: a.step(10)) == 2.0
    a.step(1)                                          # an odd number in all
    for _ in range(11):
        b.step(1)
    _same(a, b)
    a.close()
    b.close()


@pytest.mark.parametrize("case", ["clap_fling", "cylinder", "plate"])
def test_foil_and_body_force_pairs_equal_single_steps(case):
    from paper_2102_01305_amd.solver import complete_case

    bx, wg = PC.foil(case, complete_case)
    print(f"[pair] {case} with a body force", flush=True)
    a, b = _solve(bx, wg, 11, step0=210), _solve(bx, wg, 11, step0=210)
    assert _updates_per_launch(a, lambda: a.step(12)) == 2.0
    for _ in range(12):
        b.step(1)
    _same(a, b, ("u",))
    a.close()
    b.close()


def test_batch_of_first_second_and_single_steps_equals_single_steps():
    from paper_2102_01305_amd.solver import Solver, complete_case, step_batch

    print("[pair] batch with steps of all kinds", flush=True)

    def make():
        out = []
        for k, (bx, wg, storage, check, step0, alone) in enumerate(PC.batch(complete_case)):
            rng = np.random.default_rng(k)
            shape = (bx["nz"], bx["ny"], bx["nx"])
            u = rng.uniform(-5e-3, 5e-3, (3,) + shape)
            u[0] += (bx.get("u_in") or [0.0])[0]
            s = Solver(bx, wg, storage=storage, check_interval=check, history_steps=128)
            s.init_fields(rho=rng.uniform(0.995, 1.005, shape), u=u, step0=step0)
            for _ in range(alone):
                s.step(1)
            out.append(s)
        return out

    a, b = make(), make()
    step_batch(a, 70)
    for _ in range(70):
        step_batch(b, 1)
    for x, y in zip(a, b):
        print(f"[pair] batch member {x.bx['nx']}x{x.bx['ny']}x{x.bx['nz']}", flush=True)
        assert x.mass() == y.mass()
        _same(x, y, ("u", "rho"))
        if x.nw:
            n = x.step_count
            np.testing.assert_array_equal(x.forces(n - 70, 70), y.forces(n - 70, 70))
        x.close()
        y.close()
