"""Staged lists need arrays beside the plain lists: where the allocator refuses those, the
system runs on plain lists, on the same trajectory."""
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


def _run(n):
    state = gen.jitter_positions(gen.lj_fcc_state(n, gen.LJ_RHO, gen.LJ_T, n), 0.08, 3)
    sig, eps, rc = gen.lj_params()
    with make_system(state, sig, eps, rc, "sp", launch=(1, 256)) as s:
        s.set_rebuild_path(2, 2)
        s.set_integrator_nve(0.004)
        s.step(40)
        return s.get_state(), s.neighbor_pairs(), s.stats()


@pytest.mark.parametrize("refused", [1, 2, 3])
def test_plain_lists_where_the_arrays_do_not_fit(refused):
    """The refused allocation is told by its size: the 16-bit lists (half the bytes of the
    plain ones before them), the regions and the units' counts that follow."""
    import torch
    from paper_1506_05094_amd import srmd
    n = 20011
    print(f"staged arrays refused: {refused}", flush=True)
    want, pairs, stats = _run(n)
    live, sizes, hit = {}, [], [0]

    def alloc(nbytes, ctx):
        nbytes = int(nbytes)
        plain = 4 * stats["n_max"] * ((n + 63) // 64 * 64)
        first = next((k for k, b in enumerate(sizes) if 2 * b == plain), None)
        place = 1 if 2 * nbytes == plain and first is None else len(sizes) - first + 1 if first is not None else 0
        sizes.append(nbytes)
        if place == refused:
            hit[0] += 1
            return None
        t = torch.empty(max(nbytes, 1), dtype=torch.uint8, device="cuda")
        live[t.data_ptr()] = t
        return t.data_ptr()

    def free(ptr, ctx):
        live.pop(int(ptr), None)

    a, f = srmd._ALLOC_T(alloc), srmd._FREE_T(free)
    srmd._check(srmd.load().srmd_set_allocator(a, f, None))
    try:
        got, got_pairs, _ = _run(n)
    finally:
        srmd.uninstall_allocator()
    assert hit[0] == 1
    for k in ("pos", "vel", "force", "image"):
        np.testing.assert_array_equal(got[k], want[k], err_msg=k)
    np.testing.assert_array_equal(got_pairs, pairs)
