"""Run-ahead chains where lists last one step (no skin) or two: links of one and two steps
against one rebuild chain per step (step form 0), bitwise, with calls of any length, records,
and a life that grows from one step to many within a run."""
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


@pytest.mark.parametrize("skins", [(0.0,), (0.03,), (0.0, 0.3, 0.03)])
def test_short_lives(skins):
    print(f"run-ahead, skins {skins}", flush=True)
    state = gen.jitter_positions(gen.lj_fcc_state(9001, gen.LJ_RHO, 1.2, 3), 0.02, 4)
    out = []
    for form in (None, False):
        with make_system(state, *gen.lj_params(), "sp", launch=(1, 256)) as s:
            s.set_fused_reduction(form)
            s.set_integrator_nve(0.004)
            traces, builds = [], []
            for skin in skins:
                s.set_skin(skin)
                traces += [s.step(k, thermo_every=2) for k in (1, 4, 5, 60, 3, 41)]
                builds.append(s.stats()["n_rebuilds"])
            out.append((traces, s.get_state(), s.thermo(), s.stats()["steps"], builds))
    (ta, a, ra, na, ba), (tb, b, rb, nb, bb) = out
    assert na == nb == 114 * len(skins) and ba == bb and ra == rb
    for x, y in zip(ta, tb):
        assert x.tobytes() == y.tobytes()
    for k in ("pos", "vel", "force", "image"):
        np.testing.assert_array_equal(a[k], b[k])
