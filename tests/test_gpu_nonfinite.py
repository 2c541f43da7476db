"""Non-finite coordinates stay with their particles: two particles on one site turn
non-finite (r = 0) and the call reports it, the others take no contribution from them, in
every form of the force kernels; and a stateless evaluation with a NaN coordinate."""
import numpy as np
import pytest

import oracle
from workloads import generators as gen

from gpu_common import FORCE_TOL, force_error, make_system
from test_gpu_staged_potentials import lattice, salt

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
    return gen.jitter_positions(gen.lj_fcc_state(n, gen.LJ_RHO, 0.7, n), 0.05, 2), gen.lj_params(), "sp", None


def _ka(n):
    return lattice(n, gen.KA_RHO, 2, 0.6, 4), gen.ka_params(), "sf", None


def _salt(n):
    two = np.ones((2, 2))
    return lattice(n, 0.3677, 2, 1.0, 4), (two, two, 2.5 * two), "sf", salt


def _overlap(case, launch, paths):
    state, params, method, extra = case
    state = state.copy()
    state.pos[7] = state.pos[3]
    s = make_system(state, *params, method, launch=launch)
    if extra:
        extra(s)
    s.set_rebuild_path(*paths)
    s.set_integrator_nve(0.001)
    return s


def _only_these(state, what):
    for k in ("pos", "vel"):
        bad = np.nonzero(~np.isfinite(state[k]).all(axis=1))[0]
        np.testing.assert_array_equal(bad, [3, 7], err_msg=f"{what}: {k}")
    # no distance of a non-finite position is within a cutoff: no force on it either
    assert np.isfinite(state["force"]).all(), what


@pytest.mark.parametrize("case,launch,paths,persistent", [
    (lambda: _lj(864), None, (0, 0), 0), (lambda: _lj(864), (4, 64), (0, 1), 0), (lambda: _lj(864), (16, 16), (0, 1), -1),
    (lambda: _ka(1500), (1, 64), (0, 3), 0), (lambda: _lj(9001), (8, 32), (2, 3), 0), (lambda: _lj(9001), (2, 128), (2, 1), 20),
    (lambda: _lj(12007), (1, 256), (2, 2), 0), (lambda: _ka(12007), (4, 256), (2, 2), 0),
    (lambda: _salt(20011), (1, 256), (2, 2), 0), (lambda: _salt(9000), (8, 32), (2, 3), 0),
], ids=["default", "wave", "persistent", "cells", "large", "large-persistent", "staged", "staged-mixture", "staged-salt", "salt"])
def test_overlapping_pair(case, launch, paths, persistent):
    from paper_1506_05094_amd import srmd
    print(f"overlap {launch} {paths} {persistent}", flush=True)
    with _overlap(case(), launch, paths) as s:
        if persistent:
            s.set_persistent(persistent)
        with pytest.raises(srmd.SrmdError) as e:
            s.step(12)
        assert e.value.status == srmd.SRMD_ESTATE
        _only_these(s.get_state(), "after 12 steps")


def test_overlapping_pair_in_a_batch():
    from paper_1506_05094_amd import srmd
    print("overlap batch", flush=True)
    state, params, method, _ = _ka(1200)
    with _overlap(_ka(1200), (1, 256), (0, 0)) as a, make_system(state, *params, method, launch=(1, 256)) as b, \
            make_system(state, *params, method, launch=(1, 256)) as alone:
        for s in (b, alone):
            s.set_integrator_nve(0.001)
        with srmd.Batch([a, b]) as batch:
            with pytest.raises(srmd.SrmdError) as e:
                batch.step(12)
        assert e.value.status == srmd.SRMD_ESTATE
        alone.step(12)
        _only_these(a.get_state(), "batch")
        np.testing.assert_array_equal(b.get_state()["pos"], alone.get_state()["pos"])


@pytest.mark.parametrize("n", [700, 5000])
def test_stateless_forces_with_a_nan_coordinate(n):
    import torch
    from paper_1506_05094_amd import srmd
    print(f"stateless NaN {n}", flush=True)
    state, (sig, eps, rc), method, _ = _lj(n)
    pos = state.pos.copy()
    pos[5, 1] = np.nan
    pos[n // 2] = np.inf
    gone = np.array([5, n // 2])
    keep = np.setdiff1d(np.arange(n), gone).astype(np.int64)
    d_pos, d_type = torch.from_numpy(pos).cuda(), torch.from_numpy(state.types).cuda()
    force = torch.full((n, 3), 7.0, device="cuda")
    energy = torch.zeros(2, dtype=torch.float64, device="cuda")
    status = torch.full((1,), 99, dtype=torch.int32, device="cuda")
    cfg = srmd.lj_config(n, state.box, sig, eps, rc, method)
    srmd.compute_forces_noalloc(cfg, d_pos.data_ptr(), d_type.data_ptr(), force.data_ptr(), energy.data_ptr(),
                                status.data_ptr(), torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    got = force.cpu().numpy()
    assert int(status.cpu()[0]) == 0
    np.testing.assert_array_equal(got[gone], 0.0)
    ref = oracle.forces_f32(np.ascontiguousarray(state.pos[keep]), np.ascontiguousarray(state.types[keep]), state.box, sig, eps,
                            rc, method)[0]
    assert force_error(got[keep], ref) <= FORCE_TOL
    assert np.isfinite(energy.cpu().numpy()).all()
