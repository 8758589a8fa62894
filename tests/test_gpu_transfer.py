"""Checkpoint and read-back transfers: staging chunks of 2 MB (one, several,
a ragged last one; 16-bit states take the populations in more than one turn)
and force rows by kernel or by copies."""
import numpy as np
import pytest

import workloads as WL
from helpers import gpu_solver, plate

pytestmark = pytest.mark.gpu

W = np.array([1 / 3] + [1 / 18] * 6 + [1 / 36] * 12)[:, None, None, None]


def _stored(f, storage):
    """What a state of this storage holds of f, worked out in numpy."""
    v = (f - W).astype(np.float32)
    if storage == "fp16":
        return (v * np.float32(4096)).astype(np.float16).astype(np.float32) / np.float32(4096)
    if storage == "bf16":
        b = v.view(np.uint32)
        b = (b + (0x7FFF + ((b >> 16) & 1))) & np.uint32(0xFFFF0000)
        return b.astype(np.uint32).view(np.float32)
    return v


@pytest.mark.parametrize("storage", ["fp32", "fp16", "bf16"])
@pytest.mark.parametrize("size", [(4, 4, 1), (67, 35, 29), (64, 32, 256), (130, 41, 100)])
def test_checkpoint_round_trip(size, storage):
    from paper_2102_01305_amd.solver import Solver

    print(f"[transfer] {size} {storage}", flush=True)
    nx, ny, nz = size
    rng = np.random.default_rng(nx)
    f = W + rng.uniform(-2e-2, 2e-2, (19, nz, ny, nx))
    s = Solver(WL.box(nx, ny, nz, [WL.PERIODIC] * 6, 0.6), [], storage=storage)
    s.init_fields(fdist=f)
    v = _stored(f, storage)
    np.testing.assert_array_equal(s.fields("fdist"), W + v.astype(np.float64))
    # read-back of the moments: every population sits in its cell
    rho = s.fields("rho")
    want = 1.0 + sum(np.roll(v[i].astype(np.float64), (c[2], c[1], c[0]), (0, 1, 2)) for i, c in enumerate(
        [(0, 0, 0), (1, 0, 0), (-1, 0, 0), (0, 1, 0), (0, -1, 0), (0, 0, 1), (0, 0, -1), (1, 1, 0), (-1, -1, 0),
         (1, -1, 0), (-1, 1, 0), (1, 0, 1), (-1, 0, -1), (1, 0, -1), (-1, 0, 1), (0, 1, 1), (0, -1, -1), (0, 1, -1),
         (0, -1, 1)]))
    # 19 sums of values below 0.02 and their total around 1, each rounded to 32 bits
    assert np.abs(rho - want).max() <= 19 * 2.0 ** -24 * 0.4 + 2.0 ** -24
    u = s.fields("u")
    assert u.shape == (3, nz, ny, nx) and np.isfinite(u).all() and np.abs(u).max() < 0.25
    np.testing.assert_array_equal(s.fields("fdist"), W + v.astype(np.float64))   # reading changes nothing
    s.close()


@pytest.mark.parametrize("storage", ["fp32", "fp16", "bf16"])
@pytest.mark.parametrize("size", [(27, 73, 7), (69, 200, 1), (64, 32, 32), (64, 33, 32)])
def test_transfers_by_kernel_and_by_copies(size, storage):
    """Either side of the 1 MB up to which the kernels read and write host
    memory: 13797 cells of 19 values, 65536 of 4."""
    test_checkpoint_round_trip(size, storage)


@pytest.mark.parametrize("history", [7, 600, 2000])
def test_force_rows_by_kernel_and_by_copies(history):
    print(f"[transfer] force rows, ring of {history}", flush=True)
    bx, wg, ph, u0 = plate(seed=5, nz=8)
    s = gpu_solver(bx, wg, ph, u0=u0, history_steps=history)
    rows = []
    for _ in range(9):
        s.step(70)
        held = min(history, s.step_count)
        rows.append((s.step_count - held, s.forces(s.step_count - held, held)))
    first, all_rows = rows[-1]
    assert all_rows.shape[0] == min(history, 630) and np.isfinite(all_rows).all()
    for lo, part in rows:                              # 513 rows and more come by copies, fewer by kernel
        k = max(lo, first)
        np.testing.assert_array_equal(part[k - lo:], all_rows[k - first:][:max(0, lo + len(part) - k)])
    one = np.concatenate([s.forces(first + k, 1) for k in range(all_rows.shape[0])])
    np.testing.assert_array_equal(one, all_rows)
    s.close()


def test_read_back_does_not_answer_for_errors_of_other_calls():
    """An error that some other call of the thread left behind is not a failure
    of force rows or checkpoints."""
    import ctypes

    import torch  # noqa: F401  (maps the HIP runtime)

    print("[transfer] after another call's error", flush=True)
    bx, wg, ph, u0 = plate(seed=5, nz=8)
    s = gpu_solver(bx, wg, ph, u0=u0)
    s.step(3)
    f, d = s.forces(0, 3), s.fields("fdist")
    path = next(line.split()[-1] for line in open("/proc/self/maps") if "libamdhip64.so" in line)
    hip = ctypes.CDLL(path)                            # (the one already mapped)
    assert hip.hipSetDevice(1 << 20) != 0              # no such device: an error of the runtime, nothing runs
    np.testing.assert_array_equal(s.forces(0, 3), f)
    assert hip.hipSetDevice(1 << 20) != 0
    np.testing.assert_array_equal(s.fields("fdist"), d)
    hip.hipGetLastError()
    s.close()
