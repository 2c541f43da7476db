"""Staged lists (16-bit places in an LDS copy of a unit's neighbourhood; large systems with
the thread-per-particle list and whole units of 256 slots per block) against the plain
lists of the wave builder at the same layout: the same entries in the same order, so
pairs, forces and trajectories are bitwise equal.  Ragged sizes with a last unit of a
few slots, every lane count, several units per block, both fluids, the precision
variants, a box that is filled unevenly (units whose neighbourhood does not fit get plain
lists) and long flat boxes; and the readers of plain lists: pairs, saved states, the
persistent kernel."""
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


def _lj(n, seed=1):
    return gen.jitter_positions(gen.lj_fcc_state(n, gen.LJ_RHO, gen.LJ_T, n), 0.08, seed), gen.lj_params(), "sp"


def _ka(n):
    st = gen.jitter_positions(gen.lj_fcc_state(n, gen.KA_RHO, 0.6, n), 0.05, 5)
    types = np.zeros(n, np.int32)
    types[int(0.8 * n):] = 1
    types = types[np.random.default_rng(n).permutation(n)]
    return dataclasses.replace(st, types=types, ntypes=2, mass=np.array([1.0, 1.0])), gen.ka_params(), "sf"


def _uneven(n):
    """The liquid in the lower half of a box twice as high."""
    st, params, method = _lj(n)
    box = st.box * np.array([1.0, 1.0, 2.0])
    pos = st.pos.copy()
    pos[:, 2] -= np.float32(st.box[2] / 2)
    return dataclasses.replace(st, pos=gen._wrap_f32(pos, box), box=box), params, method


def _flat(n):
    """A box of 4 : 1 : 1."""
    st, params, method = _lj(4 * n)
    keep = (np.abs(st.pos[:, 1]) < st.box[1] / 4) & (np.abs(st.pos[:, 2]) < st.box[2] / 4)
    box = np.array([st.box[0], float(np.float32(st.box[1] / 2 + 0.9)), float(np.float32(st.box[2] / 2 + 0.9))])
    return dataclasses.replace(st, pos=st.pos[keep], vel=st.vel[keep], types=st.types[keep], box=box), params, method


def _system(case, launch, list_mode, precision="f32", nvt=False):
    state, (sig, eps, rc), method = case
    s = make_system(state, sig, eps, rc, method, precision=precision, launch=launch)
    s.set_rebuild_path(2, list_mode)
    s.set_integrator_nvt(0.004, 0.7, 0.2) if nvt else s.set_integrator_nve(0.004)
    return s


def _same(a, b, what):
    for k in ("pos", "vel", "force", "image", "pos64"):
        np.testing.assert_array_equal(a[k], b[k], err_msg=f"{what}: {k}")


CASES = {
    "lj4100": lambda: _lj(4100), "lj8193": lambda: _lj(8193), "lj20011": lambda: _lj(20011), "ka12345": lambda: _ka(12345),
    "uneven12000": lambda: _uneven(12000), "flat": lambda: _flat(12000),
}


@pytest.mark.parametrize("launch", [(1, 256), (2, 256), (4, 256), (1, 512), (1, 1024)])
@pytest.mark.parametrize("name", list(CASES))
def test_staged_equals_plain(name, launch):
    print(f"staged vs plain {name} {launch}", flush=True)
    case = CASES[name]()
    with _system(case, launch, 2) as a, _system(case, launch, 1) as b:
        assert a.compute_forces() == b.compute_forces()
        _same(a.get_state(), b.get_state(), "forces")
        np.testing.assert_array_equal(a.neighbor_pairs(), b.neighbor_pairs())
        a.step(41)
        b.step(41)
        _same(a.get_state(), b.get_state(), "41 steps")
        assert a.thermo() == b.thermo() and a.stats()["n_rebuilds"] == b.stats()["n_rebuilds"] > 2
        np.testing.assert_array_equal(a.neighbor_pairs(), b.neighbor_pairs())


@pytest.mark.parametrize("precision", ["f32_kahan", "f64pos"])
def test_staged_precisions(precision):
    print(f"staged {precision}", flush=True)
    case = _ka(9001)
    with _system(case, (1, 256), 2, precision, nvt=True) as a, _system(case, (1, 256), 1, precision, nvt=True) as b:
        a.step(30)
        b.step(30)
        _same(a.get_state(), b.get_state(), precision)


def test_forces_against_the_oracle():
    state, (sig, eps, rc), method = _lj(20011, 3)
    with _system((state, (sig, eps, rc), method), (1, 256), 2) as s:
        s.compute_forces()
        got = s.get_state()["force"]
    sel = np.unique(np.concatenate([np.arange(0, 20011, 41), np.argmax(np.abs(state.pos), axis=0)])).astype(np.int32)
    ref = oracle.forces_f32(state.pos, state.types, state.box, sig, eps, rc, method, sel=sel)[0]
    assert force_error(got[sel], ref) <= FORCE_TOL


def test_readers_of_plain_lists():
    """A saved state, and switches to the persistent kernel and back, between staged steps."""
    print("staged: checkpoint and persistent switches", flush=True)
    case = _lj(12007)
    with _system(case, (1, 256), 2) as a, _system(case, (1, 256), 2) as b, _system(case, (1, 256), 1) as ref:
        a.step(17)
        ref.step(17)
        blob = a.save_state()
        b.load_state(blob)
        a.step(16)
        b.step(16)
        ref.step(16)
        _same(a.get_state(), b.get_state(), "loaded")
        _same(a.get_state(), ref.get_state(), "plain")
        a.set_persistent(40)
        a.step(5)
        a.set_persistent(0)
        a.step(21)
        ref.step(26)
        _same(a.get_state(), ref.get_state(), "persistent between")
