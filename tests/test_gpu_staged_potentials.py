"""Staged lists with the potentials beside Lennard-Jones: the same entries in the same order
as the wave builder's plain lists at the same layout, so pairs, forces and steps are
bitwise equal."""
import numpy as np
import pytest

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


def lattice(n, rho, ntypes, T, seed):
    """n particles of ntypes types in turn on a jittered simple cubic lattice of density rho
    (a random subset of its sites when n does not fill it), in random order."""
    rng = np.random.default_rng(seed)
    L = float(np.float32((n / rho) ** (1.0 / 3.0)))
    box = np.array([L, L, L])
    m = int(np.ceil(n ** (1.0 / 3.0) - 1e-9))
    idx = np.stack(np.meshgrid(*[np.arange(m)] * 3, indexing="ij"), axis=-1).reshape(-1, 3)
    sites = ((idx + 0.5) * (L / m) - L / 2)[rng.permutation(m ** 3)[:n]]
    state = gen.State(pos=gen._wrap_f32(sites, box), vel=gen.maxwell_boltzmann(n, T, np.ones(n), seed).astype(np.float32),
                      types=(np.arange(n) % ntypes).astype(np.int32), box=box, mass=np.ones(ntypes), ntypes=ntypes,
                      seed=seed, recipe=f"lattice({n})")
    return gen.jitter_positions(state, 0.08, seed)


def salt(s):
    s.set_coulomb_sf([1.0, -1.0], 6.0)


def make(state, params, method, launch, extra):
    """A system with Lennard-Jones pairs (params None: what extra sets) and the extra terms."""
    import torch
    from paper_1506_05094_amd import srmd
    if params is not None:
        s = make_system(state, *params, method, launch=launch)
    else:
        s = srmd.System(state.pos, state.types, state.box, vel=state.vel, mass=state.mass, ntypes=state.ntypes,
                        stream=torch.cuda.current_stream().cuda_stream)
        s.set_skin(0.3)
        s.set_launch(*launch)
    extra(s)
    return s


def run(state, params, method, launch, list_mode, extra, steps):
    with make(state, params, method, launch, extra) as s:
        s.set_rebuild_path(2, list_mode)
        s.set_integrator_nve(0.002)
        first = s.compute_forces()
        pairs, start = s.neighbor_pairs(), s.get_state()
        s.step(steps)
        return first, pairs, start, s.get_state(), s.thermo(), s.stats()["n_rebuilds"]


def same(state, params, method, launch, extra, steps=25):
    (fa, pa, sa, a, ta, ba), (fb, pb, sb, b, tb, bb) = (
        run(state, params, method, launch, list_mode, extra, steps) for list_mode in (2, 1))
    assert fa == fb and ta == tb and ba == bb
    np.testing.assert_array_equal(pa, pb)
    for k in ("pos", "vel", "force", "image"):
        np.testing.assert_array_equal(sa[k], sb[k], err_msg=k)
        np.testing.assert_array_equal(a[k], b[k], err_msg=k)


def test_salt_at_the_largest_regions():
    """38 600 ions: regions of which the staged list kernel's LDS holds just enough places."""
    print("staged salt 38600", flush=True)
    two = np.ones((2, 2))
    same(lattice(38600, gen.SALT_RHO, 2, gen.SALT_T, 3), (two, two, 2.5 * two), "sf", (4, 256), salt, steps=12)


@pytest.mark.parametrize("launch", [(1, 256), (2, 256), (4, 256)])
def test_salt(launch):
    """Lists of about 385 entries (past the builder's ring), two cutoffs per pair."""
    print(f"staged salt {launch}", flush=True)
    two = np.ones((2, 2))
    same(lattice(20011, gen.SALT_RHO, 2, gen.SALT_T, 5), (two, two, 2.5 * two), "sf", launch, salt)


def _mie(s):
    one = np.ones((1, 1))
    s.set_pairs_mie(18 * one, 9 * one, 18 * one, 6 * one, one, 2.5 * one, "sf")


def _kind(kind, p, sigma, rc):
    def extra(s):
        one = np.ones((s.ntypes, s.ntypes))
        s.set_pairs_potential(kind, np.tile(np.asarray(p, np.float64), (s.ntypes, s.ntypes, 1)), sigma * one, rc * one, "sp")
    return extra


POTENTIALS = {
    "mie": (0.8, 1, _mie), "yukawa": (0.5, 1, _kind("yukawa", [1.3, 2.0, 0, 0], 0.9, 3.0)),
    "yukawa3": (0.5, 3, _kind("yukawa", [1.3, 2.0, 0, 0], 0.9, 3.0)),
    "gaussian": (0.5, 2, _kind("gaussian", [2.0, 0, 0, 0], 1.0, 2.6)),
    "dzugutov": (0.85, 1, _kind("dzugutov", [1.0, 0, 0, 0], 1.0, 1.94)),
}


@pytest.mark.parametrize("launch", [(1, 256), (4, 256)])
@pytest.mark.parametrize("name", list(POTENTIALS))
def test_further_potentials(name, launch):
    print(f"staged {name} {launch}", flush=True)
    rho, ntypes, extra = POTENTIALS[name]
    same(lattice(12007, rho, ntypes, 1.0, 6), None, None, launch, extra)


@pytest.mark.parametrize("launch", [(1, 256), (2, 512)])
@pytest.mark.parametrize("ntypes", [3, 4])
def test_several_types(ntypes, launch):
    """List radii of their own for every pair of three and four types (the region's copy holds
    two bits of type)."""
    print(f"staged, {ntypes} types {launch}", flush=True)
    sig = 0.8 + 0.05 * (np.arange(ntypes)[:, None] + np.arange(ntypes)[None, :])
    eps = 1.0 + 0.1 * np.abs(np.arange(ntypes)[:, None] - np.arange(ntypes)[None, :])
    same(lattice(12007, 1.0, ntypes, 1.0, 7), (sig, eps, 2.3 * sig), "sf", launch, lambda s: None)


def test_salt_against_the_oracle():
    import oracle
    oracle.load()
    print("staged salt, oracle", flush=True)
    two = np.ones((2, 2))
    state = lattice(20011, gen.SALT_RHO, 2, gen.SALT_T, 8)
    with make(state, (two, two, 2.5 * two), "sf", (1, 256), salt) as s:
        s.set_rebuild_path(2, 2)
        s.compute_forces()
        got = s.get_state()["force"]
    sel = np.unique(np.concatenate([np.arange(0, 20011, 41), np.argmax(np.abs(state.pos), axis=0)])).astype(np.int32)
    ref = oracle.forces_f32(state.pos, state.types, state.box, two, two, 2.5 * two, "sf", sel=sel, charges=[1.0, -1.0],
                            rc_coul=6.0)[0]
    assert force_error(got[sel], ref) <= FORCE_TOL
