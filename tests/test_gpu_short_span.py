"""Spans up to 16 layers, whose interpolation blocks pull their markers' band
moments themselves, at the edge of that range: against the FP64 oracle with
the bars of the parity tests, and beside a longer span in one grouped launch."""
import numpy as np
import pytest

from helpers import clap_fling, coeff_errors, gpu_solver, l2rel, oracle_sim

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nz", [4, 15, 16, 17])
def test_short_spans_against_the_oracle(nz):
    print(f"[short span] nz {nz}", flush=True)
    bx, wg, ph, u0 = clap_fling(seed=nz, nx=64, ny=48, nz=nz, chord=8.0)
    s = gpu_solver(bx, wg, ph, u0=u0, step0=90)
    o = oracle_sim(bx, wg, ph, u0=u0, step0=90)
    s.step(12)
    o.run(12)
    assert l2rel(s.fields("u"), o.fields()[1]) <= 1e-5
    assert max(coeff_errors(s.forces(90, 12), o.forces()).values()) <= 1e-3
    s.close()


@pytest.mark.parametrize("storage", ["fp32", "fp16", "bf16"])
def test_short_and_long_spans_of_one_launch(storage):
    from paper_2102_01305_amd.solver import step_batch

    print(f"[short span] batch {storage}", flush=True)
    descr = [clap_fling(seed=k, nx=64, ny=48, nz=nz, chord=8.0) for k, nz in enumerate((16, 17, 5, 40))]
    alone = [gpu_solver(bx, wg, ph, u0=u0, step0=50, storage=storage) for bx, wg, ph, u0 in descr]
    mixed = [gpu_solver(bx, wg, ph, u0=u0, step0=50, storage=storage) for bx, wg, ph, u0 in descr]
    for s in alone:
        s.step(9)
    step_batch(mixed, 9)
    for a, b in zip(alone, mixed):
        np.testing.assert_array_equal(a.forces(50, 9), b.forces(50, 9))
        np.testing.assert_array_equal(a.fields("u"), b.fields("u"))
        np.testing.assert_array_equal(a.markers("rhoB"), b.markers("rhoB"))
        a.close()
        b.close()
