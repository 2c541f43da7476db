"""A saved state holds the list entries, and zeros in the words that the control block keeps
for a running call only (a later library may use them)."""
import struct

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


@pytest.mark.parametrize("n,launch,paths", [(864, None, (0, 0)), (9001, (1, 256), (2, 2)), (9001, (8, 32), (2, 3))])
def test_words_of_a_running_call_are_zero(n, launch, paths):
    print(f"saved words {n} {paths}", flush=True)
    state = gen.jitter_positions(gen.lj_fcc_state(n, gen.LJ_RHO, 0.7, n), 0.05, 2)
    with make_system(state, *gen.lj_params(), "sp", launch=launch) as s:
        s.set_rebuild_path(*paths)
        s.set_integrator_nve(0.004)
        s.step(1)  # past the first build, before the next one
        s.step(2)
        blob, stats = bytes(s.save_state()), s.stats()
    # control block: rebuild, error, longest list, record interval, steps, builds, records,
    # trace capacity, list entries, ..., from byte 92 on the words of a running call and
    # padding, the entries once more at the end
    at = blob.index(struct.pack("<iiiiqq", 0, 0, stats["max_nbrs"], 0, 3, stats["n_rebuilds"]), 0, 1024)
    assert struct.unpack_from("<q", blob, at + 48)[0] == stats["list_entries"] > 0
    assert blob[at + 92:at + 248] == bytes(156)
