"""Staged lists in boxes with one side of more than 1024 cells: a cell is then longer than
the list radius, and the LDS copy of a unit may hold only some of a particle's own cell.
The lists, forces and steps of the thread-per-particle builder equal the wave builder's."""
import numpy as np
import pytest

from workloads import generators as gen

from gpu_common import make_system

pytestmark = pytest.mark.gpu

RC, SKIN = 2.0 ** (1.0 / 6.0), 0.1


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1506_05094_amd import srmd
    srmd.load()


def _state(cells, seed):
    """Jittered FCC lattice of the liquid's density, cells[k] unit cells along axis k."""
    a = (4.0 / gen.LJ_RHO) ** (1.0 / 3.0)
    basis = np.array([[0, 0, 0], [0, .5, .5], [.5, 0, .5], [.5, .5, 0]])
    idx = np.stack(np.meshgrid(*[np.arange(m) for m in cells], indexing="ij"), axis=-1).reshape(-1, 1, 3)
    box = np.array([float(np.float32(m * a)) for m in cells])
    sites = ((idx + basis[None] + 0.25) * a).reshape(-1, 3) - box / 2
    n = len(sites)
    sites = sites[np.random.default_rng(seed).permutation(n)]
    vel = gen.maxwell_boltzmann(n, 0.5, np.ones(n), seed).astype(np.float32)
    state = gen.State(pos=gen._wrap_f32(sites, box), vel=vel, types=np.zeros(n, np.int32), box=box, mass=np.array([1.0]),
                      ntypes=1, seed=seed, recipe=f"fcc{cells}")
    return gen.jitter_positions(state, 0.12, seed)


@pytest.mark.parametrize("cells,launch", [((4, 4, 4000), (1, 256)), ((4, 4000, 4), (4, 256)), ((4, 8000, 4), (1, 256))])
def test_long_box(cells, launch):
    print(f"long box {cells} {launch}", flush=True)
    state = _state(cells, 7)
    out = []
    for list_mode in (2, 1):
        with make_system(state, *gen.lj_params(RC), "sp", skin=SKIN, launch=launch) as s:
            s.set_rebuild_path(2, list_mode)
            s.set_integrator_nve(0.004)
            s.build_neighbor_list()
            pairs = s.neighbor_pairs()
            first = s.compute_forces()
            s.step(25)
            out.append((pairs, first, s.get_state(), s.neighbor_pairs(), s.thermo(), s.stats()["n_rebuilds"]))
    (pa, fa, a, qa, ta, ba), (pb, fb, b, qb, tb, bb) = out
    np.testing.assert_array_equal(pa, pb)
    assert fa == fb and ta == tb and ba == bb > 1
    np.testing.assert_array_equal(qa, qb)
    for k in ("pos", "vel", "force", "image"):
        np.testing.assert_array_equal(a[k], b[k], err_msg=k)
