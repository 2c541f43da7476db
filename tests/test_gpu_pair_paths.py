"""The forms of the pair loop on the GPU: one particle type (scalar constants) against a
type table with equal rows, and waves away from the box faces (no image arithmetic)
beside waves at them, at ragged sizes and lane counts whose last groups and waves are
partly idle.  Equal parameters give the same arithmetic, so the first comparison is
bitwise; the second is the force tolerance of the parity tests against the oracle."""
import dataclasses

import numpy as np
import pytest

import oracle
from workloads import generators as gen

from gpu_common import FORCE_TOL, force_error, make_system

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1506_05094_amd import srmd
    srmd.load()
    oracle.load()


@pytest.mark.parametrize("tp", [1, 4, 16, 64])
@pytest.mark.parametrize("n", [300, 4001, 12007])
@pytest.mark.parametrize("method", ["trunc", "sp", "sf"])
def test_one_type_and_interior_waves(n, tp, method):
    print(f"pair paths n={n} tp={tp} {method}", flush=True)
    state = gen.jitter_positions(gen.lj_fcc_state(n, gen.LJ_RHO, gen.LJ_T, n), 0.08, n + 1)
    sig, eps, rc = gen.lj_params()
    one = np.ones((2, 2))
    types = (np.arange(n) % 2).astype(np.int32)
    two = dataclasses.replace(state, types=types, ntypes=2, mass=np.array([1.0, 1.0]))
    forces, records = [], []
    for st, table in ((state, (sig, eps, rc)), (two, (one, one, 2.5 * one))):
        with make_system(st, *table, method, launch=(tp, 256 // tp)) as s:
            s.set_integrator_nve(0.002)
            records.append(s.compute_forces())
            forces.append(s.get_state()["force"])
            s.step(3)
            forces.append(s.get_state()["force"])
    np.testing.assert_array_equal(forces[0], forces[2])
    np.testing.assert_array_equal(forces[1], forces[3])
    assert records[0]["pe"] == records[1]["pe"] and records[0]["virial"] == records[1]["virial"]
    sel = np.unique(np.concatenate([np.arange(0, n, max(1, n // 400)), np.argmax(np.abs(state.pos), axis=0)]))
    ref = oracle.forces_f32(state.pos, state.types, state.box, sig, eps, rc, method, sel=sel.astype(np.int32))[0]
    assert force_error(forces[0][sel], ref) <= FORCE_TOL
