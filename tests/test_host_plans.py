"""The host-side rules of the launch chains (csrc/plans.h), compiled for the CPU and swept."""
import ctypes
import math
import os
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1506_05094_amd", "csrc")

SOURCE = """
#include "plans.h"
extern "C" {
void stage(int n, const double *L, const int *nc, const int *q, double reach, int tp, int ppb, int *out) {
  const srmd::StagePlan p = srmd::stage_plan(n, L, nc, q, reach, tp, ppb);
  out[0] = p.cap;
  out[1] = p.lds;
}
int slots(double life) { return srmd::ahead_slots_for(life); }
long long list_bytes(int cap) { return (long long)srmd::stage_list_bytes(cap); }
}
"""

LDS = 160 * 1024       # bytes of a compute unit
LIST_STATIC = 650      # fixed arrays of the staged list kernel
STEP_STATIC = 2400     # fixed arrays of the step kernel


@pytest.fixture(scope="module")
def plans(tmp_path_factory):
    d = tmp_path_factory.mktemp("plans")
    src, lib = str(d / "plans.cpp"), str(d / "plans.so")
    with open(src, "w") as f:
        f.write(SOURCE)
    subprocess.run(["g++", "-std=c++17", "-O1", "-shared", "-fPIC", "-I", CSRC, "-o", lib, src], check=True)
    lib = ctypes.CDLL(lib)
    lib.stage.argtypes = [ctypes.c_int] + [ctypes.c_void_p] * 3 + [ctypes.c_double] + [ctypes.c_int] * 2 + [ctypes.c_void_p]
    lib.slots.argtypes = [ctypes.c_double]
    lib.list_bytes.restype = ctypes.c_longlong
    return lib


def _stage(lib, n, rho, reach, tp, ppb, shape=(1.0, 1.0, 1.0)):
    side = (n / rho / np.prod(shape)) ** (1.0 / 3.0)
    L = np.array([side * f for f in shape])
    nc = np.array([max(1, min(int(l / (0.5 * reach * (1 + 1e-5))), 1024)) for l in L], np.int32)
    q = np.array([c // max(1, c // 5) for c in nc[:2]], np.int32)
    out = np.zeros(2, np.int32)
    lib.stage(n, L.ctypes.data, nc.ctypes.data, q.ctypes.data, reach, tp, ppb, out.ctypes.data)
    return int(out[0]), int(out[1])


@pytest.mark.parametrize("tp,ppb", [(1, 256), (2, 256), (4, 256), (1, 512), (2, 512), (1, 1024)])
def test_staged_launches_fit_the_lds(plans, tp, ppb):
    """Wherever the rule takes staged lists, the list kernel and the step kernel both fit a
    compute unit, and the capacity is at least 1024 places."""
    taken = 0
    for rho in (0.05, 0.3677, 0.8442, 1.2, 3.0):
        for reach in np.concatenate([np.arange(0.8, 4.0, 0.2), np.arange(4.0, 9.0, 0.05)]):
            for n in np.unique(np.geomspace(8193, 4e6, 40).astype(int)):
                cap, lds = _stage(plans, int(n), rho, float(reach), tp, ppb)
                if cap == 0:
                    continue
                taken += 1
                what = (rho, reach, n, cap, lds)
                assert plans.list_bytes(cap) + LIST_STATIC <= LDS, what
                assert 16 * lds + STEP_STATIC <= LDS and lds == ppb // 256 * (cap + 1) and cap >= 1024, what
    assert taken > 100


def test_regions_at_the_edge_stay_staged(plans):
    """The salt of 38 600 at four lanes per particle: its capacity would be past what the list
    kernel has room for."""
    cap, _ = _stage(plans, 38600, 0.3677, 6.3, 4, 256)
    assert 8900 < cap and plans.list_bytes(cap) + LIST_STATIC <= LDS


@pytest.mark.parametrize("n", [64000, 256000, 1024000])
def test_the_liquid_keeps_five_blocks_per_compute_unit(plans, n):
    cap, lds = _stage(plans, n, 0.8442, 2.8, 1, 256)
    assert 0 < cap <= 1850 and 16 * lds + STEP_STATIC <= LDS // 5


def test_other_layouts_and_small_grids_take_plain_lists(plans):
    assert _stage(plans, 64000, 0.8442, 2.8, 1, 128)[0] == 0
    assert _stage(plans, 1500, 0.8442, 2.8, 1, 256)[0] == 0
    assert math.prod(_stage(plans, 1 << 28, 0.8442, 2.8, 1, 256)) == 0


IDLE_REBUILD, IDLE_STEP = 7.5, 1.5  # us of a rebuild slot that is not due, of a step that waits for one


def _idle(life, slots):
    """Idle time per rebuild at a whole number of steps per list."""
    links = -(-life // slots)
    return (links - 1) * IDLE_REBUILD + (links * slots - life) * IDLE_STEP


def test_run_ahead_slots_cost_no_more_than_a_slot_per_step(plans):
    """For any list life, also one that varies by a step, run-ahead chains idle no longer than
    a rebuild slot before every step does, and not much longer than the best of the counts."""
    for whole in range(1, 60):
        for part in (0.0, 0.25, 0.5, 0.75):
            k = plans.slots(whole + part)
            idle = lambda s: (1 - part) * _idle(whole, s) + part * _idle(whole + 1, s)
            assert idle(k) <= (1 - part) * (whole - 1) * IDLE_REBUILD + part * whole * IDLE_REBUILD + 1e-9, (whole, part, k)
            if whole < 3:
                assert idle(k) <= 1.25 * min(idle(s) for s in (1, 2, 8)) + 1.0, (whole, part, k)

