"""Run-ahead chains (large systems: rebuild slots and the steps between them, the count of
steps kept on the device) against one rebuild chain per step (step form 0): calls of any
length, lists that last two steps, about ten or the whole run, records and counters;
also after an overflow replay.  Bitwise equal."""
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


CALLS = [1, 3, 4, 5, 40, 2, 97, 8, 1]


@pytest.mark.parametrize("skin,T", [(0.06, 1.5), (0.3, 0.7), (0.9, 0.01)])
@pytest.mark.parametrize("list_mode,launch", [(2, (1, 256)), (3, (8, 32))])
def test_ahead_equals_per_step_chain(list_mode, launch, skin, T):
    print(f"run-ahead skin={skin} mode={list_mode} launch={launch}", flush=True)
    state = gen.jitter_positions(gen.lj_fcc_state(9001, gen.LJ_RHO, T, 3), 0.02, 4)
    out = []
    for form in (None, False):
        with make_system(state, *gen.lj_params(), "sp", skin=skin, launch=launch) as s:
            s.set_rebuild_path(2, list_mode)
            s.set_fused_reduction(form)
            s.set_integrator_nvt(0.004, max(T, 0.01), 0.2)
            traces = [s.step(k, thermo_every=3) for k in CALLS]
            out.append((traces, s.get_state(), s.thermo(), s.stats()["steps"], s.stats()["n_rebuilds"]))
    (ta, a, ra, na, ba), (tb, b, rb, nb, bb) = out
    assert na == nb == sum(CALLS) and ba == bb >= 1 and ra == rb
    for x, y in zip(ta, tb):
        assert x.tobytes() == y.tobytes()
    for k in ("pos", "vel", "force", "image"):
        np.testing.assert_array_equal(a[k], b[k])


def test_switches_between_forms():
    """Calls in the run-ahead, per-step and persistent forms after each other."""
    state = gen.jitter_positions(gen.lj_fcc_state(9001, gen.LJ_RHO, gen.LJ_T, 3), 0.05, 4)
    with make_system(state, *gen.lj_params(), "sp", launch=(2, 128)) as s, \
            make_system(state, *gen.lj_params(), "sp", launch=(2, 128)) as ref:
        ref.set_fused_reduction(False)
        for x in (s, ref):
            x.set_integrator_nve(0.004)
        s.step(23)
        s.set_persistent(30)
        s.step(9)
        s.set_persistent(0)
        s.step(14)
        s.set_fused_reduction(False)
        s.step(5)
        s.set_fused_reduction(None)
        s.step(30)
        ref.step(46)
        ref.set_fused_reduction(False)  # choosing a form requests a list build
        ref.step(5)
        ref.set_fused_reduction(False)
        ref.step(30)
        a, b = s.get_state(), ref.get_state()
        for k in ("pos", "vel", "force", "image"):
            np.testing.assert_array_equal(a[k], b[k])
        assert s.thermo() == ref.thermo()
