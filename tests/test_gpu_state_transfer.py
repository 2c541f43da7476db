"""State transfers in original particle order: what srmd_set_state puts in comes back
from srmd_get_state exactly, whatever order the device keeps the particles in, for the
transfers through pinned memory and (from 116 509 particles on) direct ones."""
import ctypes

import numpy as np
import pytest

from workloads import generators as gen

from gpu_common import make_system

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1506_05094_amd import srmd
    srmd.load()


@pytest.mark.parametrize("precision", ["f32", "f32_kahan", "f64pos"])
@pytest.mark.parametrize("n", [257, 20011, 116508, 116509])
def test_round_trip(n, precision):
    print(f"state transfer n={n} {precision}", flush=True)
    from paper_1506_05094_amd import srmd

    state = gen.lj_fcc_state(n, gen.LJ_RHO, gen.LJ_T, n)
    rng = np.random.default_rng(n)
    half = state.box[0] / 2
    with make_system(state, *gen.lj_params(), "sp", precision=precision) as s:
        s.set_integrator_nve(0.002)
        s.step(5)  # the device order is now the sorted one
        before = s.get_state()
        # velocities alone: positions stay, bit for bit
        vel = rng.standard_normal((n, 3)).astype(np.float32)
        s.set_state(vel=vel)
        got = s.get_state()
        np.testing.assert_array_equal(got["vel"], vel)
        np.testing.assert_array_equal(got["pos"], before["pos"])
        # positions outside the box come back wrapped, images cleared, velocities kept
        shift = rng.integers(-2, 3, size=(n, 3))
        s.step(3)
        kept = s.get_state()["vel"]
        far = (state.pos.astype(np.float64) + shift * state.box).astype(np.float32)
        s.set_state(pos=far)
        got = s.get_state()
        want = far.astype(np.float64) - state.box * np.floor(far.astype(np.float64) / state.box + 0.5)
        want = want.astype(np.float32)
        want[want >= np.float32(half)] -= np.float32(state.box[0])
        np.testing.assert_array_equal(got["pos"], want)
        np.testing.assert_array_equal(got["pos64"], want.astype(np.float64))
        np.testing.assert_array_equal(got["vel"], kept)
        assert not got["image"].any()
        # any subset of the arrays
        only = np.zeros((n, 3), np.int32)
        srmd.srmd_get_state(s._h, None, None, only.ctypes.data_as(ctypes.POINTER(ctypes.c_int32)), None, None)
        assert not only.any()
        # a refused state changes nothing
        bad = state.pos.copy()
        bad[n // 2, 1] = np.nan
        with pytest.raises(srmd.SrmdError):
            s.set_state(pos=bad, vel=vel)
        again = s.get_state()
        np.testing.assert_array_equal(again["pos"], got["pos"])
        np.testing.assert_array_equal(again["vel"], got["vel"])
