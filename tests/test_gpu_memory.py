"""Refused device memory: what a system does without its optional arrays."""
import contextlib

import numpy as np
import pytest

from workloads import generators as gen

from gpu_common import make_system

pytestmark = pytest.mark.gpu

N = 20011


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1506_05094_amd import srmd
    srmd.load()


class Hook:
    """Allocations through torch; refuse(sizes so far, bytes) says which fail."""

    def __init__(self):
        self.sizes, self.live, self.refused, self.refuse = [], {}, [], lambda sizes, nbytes: False

    def alloc(self, nbytes, ctx):
        import torch
        nbytes = int(nbytes)
        if self.refuse(self.sizes, nbytes):
            self.refused.append(nbytes)
            return None
        self.sizes.append(nbytes)
        t = torch.empty(max(nbytes, 1), dtype=torch.uint8, device="cuda")
        self.live[t.data_ptr()] = t
        return t.data_ptr()

    def free(self, ptr, ctx):
        self.live.pop(int(ptr), None)

    def held(self):
        return sum(t.numel() for t in self.live.values())


@contextlib.contextmanager
def hooked():
    from paper_1506_05094_amd import srmd
    h = Hook()
    a, f = srmd._ALLOC_T(h.alloc), srmd._FREE_T(h.free)
    srmd._check(srmd.load().srmd_set_allocator(a, f, None))
    try:
        yield h
    finally:
        srmd.uninstall_allocator()


def _state(n=N):
    return gen.jitter_positions(gen.lj_fcc_state(n, gen.LJ_RHO, gen.LJ_T, n), 0.08, 3)


def _liquid(state, launch=(1, 256), list_mode=0, precision="f32"):
    s = make_system(state, *gen.lj_params(), "sp", launch=launch, precision=precision)
    s.set_rebuild_path(0, list_mode)
    s.set_integrator_nve(0.004)
    return s


def test_automatic_builder_without_the_staged_arrays():
    """Where the staged lists' arrays are refused, the automatic choice is that of a system
    without staged lists: the cell builder up to 131072 particles."""
    print("automatic builder, staged arrays refused", flush=True)
    with _liquid(_state()) as s:
        s.step(20)
        want, stats = s.get_state(), s.stats()
        plain = 4 * stats["n_max"] * ((N + 63) // 64 * 64)
    assert stats["list_mode"] == 2
    with hooked() as h:
        h.refuse = lambda sizes, nbytes: plain in sizes and 2 * nbytes == plain  # the 16-bit lists
        with _liquid(_state()) as s:
            s.step(20)
            got, stats = s.get_state(), s.stats()
    assert h.refused and stats["list_mode"] == 3
    for k in ("pos", "vel", "force", "image"):
        np.testing.assert_array_equal(got[k], want[k], err_msg=k)


def _uneven():
    """The liquid in the lower half of a box twice as high: its lists outgrow the first capacity."""
    st = _state()
    box = st.box * np.array([1.0, 1.0, 2.0])
    pos = st.pos.copy()
    pos[:, 2] -= np.float32(st.box[2] / 2)
    return gen.State(pos=gen._wrap_f32(pos, box), vel=st.vel, types=st.types, box=box, mass=st.mass, ntypes=1, seed=st.seed,
                     recipe=st.recipe)


def _run(state, list_mode, precision, h):
    """Two calls, the second with records; what the system then holds, and the results."""
    with _liquid(state, list_mode=list_mode, precision=precision) as s:
        s.step(15)
        trace = s.step(20, thermo_every=1)
        held = h.held()
        h.refuse = lambda sizes, nbytes: False
        return held, (trace, s.get_state(), s.neighbor_pairs(), s.stats()["n_max"])


@pytest.mark.parametrize("just_short", [False, True])
@pytest.mark.parametrize("name,state,precision", [("even", _state, "f32"), ("uneven", _uneven, "f32"),
                                                  ("f64pos", _state, "f64pos")])
def test_steps_in_less_memory(name, state, precision, just_short):
    """Under a budget of what the wave builder's plain lists hold in the end (arrays, snapshot,
    trace, a list that grew), and of one byte less than staged lists do: they give their
    arrays back instead of failing the call, on the same trajectory."""
    print(f"memory: {name}, just short of the staged lists' {just_short}", flush=True)
    with hooked() as h:
        budget, want = _run(state(), 1, precision, h)
        if just_short:
            budget = _run(state(), 2, precision, h)[0] - 1
    with hooked() as h:
        h.refuse = lambda sizes, nbytes: h.held() + nbytes > budget
        held, got = _run(state(), 2, precision, h)
        assert h.refused and held <= budget
    assert got[0].tobytes() == want[0].tobytes() and got[3] == want[3]
    np.testing.assert_array_equal(got[2], want[2])
    for k in ("pos", "vel", "force", "image", "pos64"):
        np.testing.assert_array_equal(got[1][k], want[1][k], err_msg=k)


def test_a_smaller_trace_after_a_refused_one():
    """A trace buffer that could not grow leaves none behind: the next call makes its own."""
    from paper_1506_05094_amd import srmd
    print("refused trace", flush=True)
    with hooked() as h, _liquid(_state(), list_mode=1) as s:
        s.step(8, thermo_every=1)
        h.refuse = lambda sizes, nbytes: nbytes > 10 * 1024
        with pytest.raises(srmd.SrmdError) as e:
            s.step(1000, thermo_every=1)
        assert e.value.status == srmd.SRMD_ENOMEM
        assert len(s.step(4, thermo_every=1)) == 4 and s.stats()["steps"] == 12


@pytest.mark.parametrize("n,precision", [(700, "f32"), (700, "f64pos"), (9001, "f32_kahan"), (9001, "f64pos"), (130001, "f32")])
def test_state_transfers_without_device_memory(n, precision):
    """With every further allocation refused, states are read and set as with the transfer
    buffer, a new state with and without positions or velocities."""
    print(f"state transfers, no device memory: {n} {precision}", flush=True)
    state = _state(n)
    rng = np.random.default_rng(n)
    pos = (state.pos + 3.0 * rng.standard_normal((n, 3))).astype(np.float32)  # past the faces: wrapped
    vel = rng.standard_normal((n, 3)).astype(np.float32)
    out = []
    for refused in (False, True):
        with hooked() as h, _liquid(state, launch=(1, 64), list_mode=1, precision=precision) as s:
            s.step(5)
            h.refuse = lambda sizes, nbytes: refused
            seen = [s.get_state()]
            for new in (dict(vel=vel), dict(pos=state.pos), dict(pos=pos, vel=vel)):
                s.set_state(**new)
                seen.append(s.get_state())
            s.set_state(pos=state.pos, vel=state.vel)
            s.step(5)
            seen.append(s.get_state())
            assert bool(h.refused) == refused
            out.append(seen)
    for k, (a, b) in enumerate(zip(*out)):
        for key in a:
            np.testing.assert_array_equal(a[key], b[key], err_msg=f"{k}: {key}")


@pytest.mark.parametrize("n,kept", [(20000, True), (3_800_000, False)])
def test_large_transfer_buffers_are_given_back(n, kept):
    """The transfer buffer (72 bytes per particle) stays up to 256 MiB; a larger one does not."""
    from paper_1506_05094_amd import srmd
    print(f"transfer buffer of {n}", flush=True)
    L = float(np.float32((n / gen.LJ_RHO) ** (1.0 / 3.0)))
    pos = np.random.default_rng(n).uniform(-0.499 * L, 0.499 * L, (n, 3)).astype(np.float32)
    with hooked() as h, srmd.System(pos, np.zeros(n, np.int32), [L] * 3, vel=pos) as s:
        before = h.held()
        np.testing.assert_array_equal(s.get_state()["pos"], pos)
        assert (h.held() > before) == kept
        s.set_state(pos=pos[::-1].copy())
        assert (h.held() > before) == kept
        got = s.get_state()
        np.testing.assert_array_equal(got["pos"], pos[::-1])
        np.testing.assert_array_equal(got["vel"], pos)


def test_readers_after_a_refused_layout():
    """A change to staged lists whose cell arrays are refused leaves constants without arrays:
    the readers of lists touch none of them, and the next call makes the layout."""
    from paper_1506_05094_amd import srmd
    print("refused layout, then readers", flush=True)
    with hooked() as h, _liquid(_state(), launch=(8, 32), list_mode=3) as s, \
            _liquid(_state(), launch=(1, 256), list_mode=1) as ref:
        s.step(5)
        s.set_launch(1, 256)
        s.set_rebuild_path(2, 2)
        s.set_skin(0.1)  # more cells: their arrays are made anew
        h.refuse = lambda sizes, nbytes: True
        for call in (lambda: s.step(5), s.save_state, s.compute_forces):
            with pytest.raises(srmd.SrmdError) as e:
                call()
            assert e.value.status == srmd.SRMD_ENOMEM
        with contextlib.suppress(srmd.SrmdError):
            s.neighbor_pairs()
        h.refuse = lambda sizes, nbytes: False
        start = s.get_state()
        s.step(10)
        ref.set_skin(0.1)
        ref.set_state(pos=start["pos"], vel=start["vel"])
        s.set_state(pos=start["pos"], vel=start["vel"])
        s.step(10)
        ref.step(10)
        np.testing.assert_array_equal(s.neighbor_pairs(), ref.neighbor_pairs())
        a, b = s.get_state(), ref.get_state()
        for k in ("pos", "vel", "force"):
            np.testing.assert_array_equal(a[k], b[k], err_msg=k)


def test_fewer_groups_after_a_refused_job_table():
    """A persistent job table that could not grow leaves none behind either."""
    from paper_1506_05094_amd import srmd
    print("refused job table", flush=True)
    state = _state(2000)
    with hooked() as h, _liquid(state, launch=(8, 32)) as s, _liquid(state, launch=(8, 32)) as ref:
        s.set_persistent(4)
        s.step(3)
        s.set_persistent(40)
        h.refuse = lambda sizes, nbytes: nbytes == 40 * 16  # the table of 40 jobs
        with pytest.raises(srmd.SrmdError) as e:
            s.step(3)
        assert h.refused and e.value.status == srmd.SRMD_ENOMEM
        s.set_persistent(3)
        s.step(3)
        ref.step(6)
        np.testing.assert_array_equal(s.get_state()["pos"], ref.get_state()["pos"])
