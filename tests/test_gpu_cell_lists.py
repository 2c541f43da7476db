"""Cell lists (a wave per piece of a cell; in a batch by rounds of 128 slots staged in LDS)
against the lists of one wave per particle: the same entries in the same order, so pairs and
trajectories are bitwise equal.  Systems below and above 7 cells per axis (image arithmetic
per pair, or from the cells), a last round or workgroup of a few slots, crowded and empty
cells, lists longer than the LDS stage, one to three types, and replicas whose sorted
positions fit in LDS beside the stage or not."""
import dataclasses

import numpy as np
import pytest

import oracle
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
    oracle.load()


def _lj(n):
    return gen.jitter_positions(gen.lj_fcc_state(n, gen.LJ_RHO, gen.LJ_T, n), 0.08, n), gen.lj_params(), "sp"


def _ka(n):
    return gen.ka_random_state(n, 1.2, 0.7, n), gen.ka_params(), "sf"


def _three(n):
    """Three types with cutoffs of their own."""
    st, _, _ = _lj(n)
    types = np.random.default_rng(n).integers(0, 3, n).astype(np.int32)
    sig = np.array([[1.0, 0.95, 0.9], [0.95, 0.9, 0.85], [0.9, 0.85, 0.8]])
    return dataclasses.replace(st, types=types, ntypes=3, mass=np.ones(3)), (sig, np.ones((3, 3)), 2.5 * sig), "sf"


def _dense(n):
    """Cutoff 3.2: lists of more than 128 entries."""
    st, (sig, eps, _), method = _ka(n)
    return st, (sig, eps, np.full((2, 2), 3.2)), method


def _uneven(n):
    """The liquid in the lower half of a box twice as high: empty cells."""
    st, params, method = _lj(n)
    box = st.box * np.array([1.0, 1.0, 2.0])
    pos = st.pos.copy()
    pos[:, 2] -= np.float32(st.box[2] / 2)
    return dataclasses.replace(st, pos=gen._wrap_f32(pos, box), box=box), params, method


KINDS = {"lj": _lj, "ka": _ka, "three": _three, "dense": _dense, "uneven": _uneven}


def _system(case, launch, list_mode=0):
    state, (sig, eps, rc), method = case
    s = make_system(state, sig, eps, rc, method, launch=launch)
    if list_mode:
        s.set_rebuild_path(0, list_mode)
    s.set_integrator_nve(0.003)
    return s


def _same(a, b, what):
    x, y = a.get_state(), b.get_state()
    for k in ("pos", "vel", "force", "image"):
        np.testing.assert_array_equal(x[k], y[k], err_msg=f"{what}: {k}")


@pytest.mark.parametrize("launch", [(1, 128), (8, 32)])
@pytest.mark.parametrize("kind,n", [("lj", 1001), ("lj", 4129), ("lj", 9000), ("ka", 700), ("ka", 5003), ("three", 3007),
                                    ("dense", 4001), ("uneven", 2500)])
def test_cell_lists_equal_wave_lists(kind, n, launch):
    print(f"cell lists {kind} {n} {launch}", flush=True)
    case = KINDS[kind](n)
    with _system(case, launch, 3) as a, _system(case, launch, 1) as b:
        a.compute_forces()
        b.compute_forces()
        np.testing.assert_array_equal(a.neighbor_pairs(), b.neighbor_pairs())
        a.step(40)
        b.step(40)
        assert a.stats()["n_rebuilds"] == b.stats()["n_rebuilds"] > 1
        _same(a, b, f"{kind} {n} {launch}")


@pytest.mark.parametrize("launch,groups", [((1, 256), 4), ((1, 256), 0), ((2, 128), 5), ((4, 64), 4), ((8, 32), 6)])
@pytest.mark.parametrize("kind,sizes", [("ka", (641, 1900, 5200, 8192)), ("lj", (1025, 2177, 6001, 7900)),
                                        ("three", (900, 2300, 3007, 4200)), ("dense", (2000, 2501, 4001, 5300))])
def test_batch_rounds_equal_wave_lists(kind, sizes, launch, groups):
    """Whole replicas on a workgroup, replicas split over a few, and (groups 0) over so many
    that each wave takes particles one by one, against each replica's own launch chain."""
    from paper_1506_05094_amd import srmd
    print(f"batch lists {kind} {launch} max_workgroups={groups}", flush=True)
    cases = [KINDS[kind](n) for n in sizes]
    single = [_system(c, launch, 1) for c in cases]
    batched = [_system(c, launch) for c in cases]
    for s in single:
        s.step(40)
    with srmd.Batch(batched, max_workgroups=groups) as b:
        b.step(40)
    for a, c, n in zip(single, batched, sizes):
        assert a.stats()["n_rebuilds"] == c.stats()["n_rebuilds"] > 1
        assert a.stats()["max_nbrs"] == c.stats()["max_nbrs"]
        _same(a, c, f"{kind} {n} {launch} {groups}")
    for s in single + batched:
        s.close()
