"""The allocation-free force entry at sizes around its workgroups, against the allocating path
at the same default launch shape (bit for bit): positions outside the box, a type out of
range, and the launches in a captured graph that is replayed on changing positions."""
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


class _Direct:
    def __init__(self, state, params, method):
        import torch
        from paper_1506_05094_amd import srmd
        n = state.n
        self.pos = torch.from_numpy(np.ascontiguousarray(state.pos, np.float32)).cuda()
        self.types = torch.from_numpy(np.ascontiguousarray(state.types, np.int32)).cuda()
        self.force = torch.full((n, 3), float("nan"), device="cuda")
        self.energy = torch.full((2,), float("nan"), dtype=torch.float64, device="cuda")
        self.status = torch.full((1,), -1, dtype=torch.int32, device="cuda")
        self.cfg = srmd.lj_config(n, state.box, *params, method, 0.3)

    def __call__(self):
        import torch
        from paper_1506_05094_amd import srmd
        srmd.compute_forces_noalloc(self.cfg, self.pos.data_ptr(), self.types.data_ptr(), self.force.data_ptr(),
                                    self.energy.data_ptr(), self.status.data_ptr(),
                                    torch.cuda.current_stream().cuda_stream)

    def result(self):
        return self.force.cpu().numpy(), self.energy.cpu().numpy(), int(self.status.cpu().item())


def _allocating(state, params, method):
    with make_system(state, *params, method, skin=0.3) as s:
        th = s.compute_forces()
        return s.get_state()["force"], np.array([th["pe"], th["virial"]])


def _state(kind, n):
    if kind == "ka":
        return gen.ka_random_state(n, 1.2, 0.7, n), gen.ka_params(), "sf"
    return gen.jitter_positions(gen.lj_fcc_state(n, gen.LJ_RHO, gen.LJ_T, n), 0.08, n), gen.lj_params(), "sp"


@pytest.mark.parametrize("kind,n", [("lj", 500), ("lj", 1023), ("lj", 1025), ("ka", 1500), ("ka", 4095), ("lj", 4097),
                                    ("ka", 8192)])
def test_direct_equals_allocating(kind, n):
    print(f"direct {kind} {n}", flush=True)
    state, params, method = _state(kind, n)
    want_f, want_e = _allocating(state, params, method)
    d = _Direct(state, params, method)
    d()
    f, e, status = d.result()
    assert status == 0
    np.testing.assert_array_equal(f, want_f)
    np.testing.assert_array_equal(e, want_e)


def test_direct_reports_a_type_out_of_range():
    state, params, method = _state("ka", 1025)
    state.types[:] = np.where(np.arange(1025) == 1024, 0, state.types)
    want_f, want_e = _allocating(state, params, method)
    d = _Direct(state, params, method)
    d.types[1024] = 7  # taken as type 0
    d()
    f, e, status = d.result()
    assert status == 4
    np.testing.assert_array_equal(f, want_f)
    np.testing.assert_array_equal(e, want_e)


def test_direct_in_a_graph():
    import torch
    state, params, method = _state("lj", 1025)
    d = _Direct(state, params, method)
    d()
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        d()
    base = d.pos.clone()
    for k in range(4):
        print(f"direct graph replay {k}", flush=True)
        d.pos.copy_(base + 0.02 * k * torch.sin(torch.arange(3 * 1025, device="cuda").reshape(1025, 3).float()))
        graph.replay()
        torch.cuda.synchronize()
        got = d.result()
        d.force.fill_(float("nan"))
        d()
        torch.cuda.synchronize()
        want = d.result()
        assert got[2] == want[2] == 0
        np.testing.assert_array_equal(got[0], want[0])
        np.testing.assert_array_equal(got[1], want[1])
