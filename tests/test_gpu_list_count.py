"""The entry count of the current list: equal to its pairs for every builder, carried by a
saved state, and read from a state that holds it only in its older place."""
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


def _system(n, launch, list_mode):
    state = gen.jitter_positions(gen.lj_fcc_state(n, gen.LJ_RHO, gen.LJ_T, n), 0.08, n)
    sig, eps, rc = gen.lj_params()
    s = make_system(state, sig, eps, rc, "sp", launch=launch)
    s.set_rebuild_path(0, list_mode)
    s.set_integrator_nve(0.004)
    return s


@pytest.mark.parametrize("n,launch,list_mode", [(1001, (32, 8), 1), (1001, (8, 32), 4), (4129, (8, 32), 3),
                                                (9001, (1, 256), 2), (9001, (4, 64), 5)])
def test_entry_count(n, launch, list_mode):
    print(f"entry count {n} {launch} mode {list_mode}", flush=True)
    with _system(n, launch, list_mode) as a, _system(n, launch, list_mode) as b, _system(n, launch, list_mode) as c:
        a.step(23)
        a.compute_forces()  # a list for the positions of now, where a build was due
        count = a.stats()["list_entries"]
        assert count == len(a.neighbor_pairs()) > 0
        blob = bytearray(a.save_state())
        b.load_state(bytes(blob))
        assert b.stats()["list_entries"] == count
        words = np.frombuffer(bytes(blob[:1024]), np.int64)
        places = np.nonzero(words == count)[0]
        assert len(places) == 2
        blob[8 * places[1]:8 * places[1] + 8] = bytes(8)
        c.load_state(bytes(blob))
        assert c.stats()["list_entries"] == count
