"""Staged lists with the potentials beside Lennard-Jones: the same entries in the same order
as the wave builder's plain lists at the same layout, so pairs, forces and steps are
bitwise equal."""
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


def run(state, params, method, launch, list_mode, extra, steps):
    with make_system(state, *params, method, launch=launch) as s:
        extra(s)
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
