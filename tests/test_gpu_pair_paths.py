"""Two steps in one pass against the same steps one by one, bit for bit, where
a block's column is ragged and on the paths that only some solves take: a last
column of one cell, a last tile of one row, foils with a body force.
test_host_api.py checks on the CPU that these solves are planned in pairs."""
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
