"""The work a user of srmd has it do, as cases that can be timed and checked.

A case is a dict of plain values; its "kind" says which calls a pass makes:

* "steps"    a production block of one system: ``System.step`` and the frame that a
             program writes after it (``System.get_state``);
* "batch"    the same for many independent replicas advanced together;
* "forces"   energies and forces of a new configuration: ``System.set_state``,
             ``System.compute_forces``, ``System.get_state``;
* "noalloc"  forces of a configuration in device memory, with no allocation and no
             host synchronisation (``compute_forces_noalloc``).

Fluids: the single-component Lennard-Jones liquid (shifted potential, NVE, a melting
FCC start), the Kob-Andersen mixture (shifted force, Nose-Hoover NVT) and the molten
salt with shifted-force Coulomb (NVT).  "tuned" 0 runs the library's default layout,
1 a layout as the autotuner picks it for that size.
"""
import math

import numpy as np
import torch

from paper_1506_05094_amd import srmd

# per fluid: density, start temperature, time step, list reach and force reach (sigma)
FLUIDS = {
    "lj": dict(rho=0.8442, T=1.44, dt=0.005, jitter=0.05),
    "ka": dict(rho=1.2, T=0.45, dt=0.005, jitter=0.04),
    "salt": dict(rho=0.3677, T=2.0, dt=0.004, jitter=0.10),
}
SKIN = 0.3
TAU = 0.2
RC_COULOMB = 6.0
# mean list entries and in-range partners per particle at these densities and skin 0.3
PARTNERS = {"lj": (77.6, 55.3), "ka": (91.9, 63.8), "salt": (385.0, 333.0)}
# float operations of a listed pair's distance test and of an in-range pair
OPS = {"lj": (20, 21), "ka": (20, 27), "salt": (20, 40)}


def _steps(name, fluid, n, steps, tuned=0, precision="f32"):
    return dict(name=name, kind="steps", fluid=fluid, n=n, steps=steps, tuned=tuned, precision=precision)


def listed():
    return [
        # force evaluation inside a host program's own loop, device memory in and out
        dict(name="noalloc_lj_1500", kind="noalloc", fluid="lj", n=1500),
        # the smallest system of the size sweep: launch latency and nothing else
        _steps("steps_lj_864", "lj", 864, 100),
        # the headline workload, at the autotuner's layout
        _steps("steps_ka_4096", "ka", 4096, 100, tuned=1),
        # a ragged size at the default layout, just past the largest one-launch step
        _steps("steps_ka_5003", "ka", 5003, 100),
        # sizes of the sweep between "a few thousand" and "fills the chip"
        _steps("steps_lj_16000", "lj", 16000, 100, tuned=1),
        # the precision study: float64 master positions
        _steps("steps_lj_32768_f64", "lj", 32768, 100, precision="f64pos"),
        _steps("steps_lj_64000", "lj", 64000, 100, tuned=1),
        _steps("steps_lj_256000", "lj", 256000, 100, tuned=1),
        # the size sweep's largest, at the default layout
        _steps("steps_lj_1024000", "lj", 1024000, 100),
        # the Coulomb benchmark: lists five times longer
        _steps("steps_salt_20000", "salt", 20000, 100),
        # the replica set: many uneven small systems in one launch
        dict(name="batch_ka_256", kind="batch", fluid="ka", replicas=256, lo=500, hi=8000, steps=200),
        # energies of new configurations (minimisers, Monte Carlo): sort, list, forces
        dict(name="forces_lj_64000", kind="forces", fluid="lj", n=64000),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["steps", "steps", "steps", "steps", "batch", "forces", "noalloc"])
    if kind == "noalloc":
        return dict(kind=kind, fluid=rng.choice(["lj", "ka"]), n=_log_int(rng, 500, 8000))
    if kind == "forces":
        return dict(kind=kind, fluid=rng.choice(["lj", "ka"]), n=_log_int(rng, 1000, 500000))
    if kind == "batch":
        lo = _log_int(rng, 400, 1500)
        return dict(kind=kind, fluid="ka", replicas=_log_int(rng, 8, 200), lo=lo, hi=rng.randint(3 * lo, 8000),
                    steps=rng.randint(50, 200))
    fluid = rng.choice(["lj", "lj", "ka", "salt"])
    n = _log_int(rng, 2000, 100000) // 2 * 2 if fluid == "salt" else _log_int(rng, 700, 1000000)
    precision = rng.choice(["f32", "f32", "f32", "f32_kahan", "f64pos"])
    return dict(kind="steps", fluid=fluid, n=n, steps=rng.randint(60, 100), tuned=rng.randint(0, 1),
                precision=precision)


# ---------------------------------------------------------------- inputs


def _side(n, rho):
    return float(np.float32((n / rho) ** (1.0 / 3.0)))


def _start(fluid, n, rng, T=None):
    """Positions float32 in [-L/2, L/2), velocities float32, types int32, box side: a
    jittered lattice of the fluid's density (FCC, simple cubic for the salt; a random
    subset of its sites when n does not fill it) and Maxwell-Boltzmann velocities."""
    f = FLUIDS[fluid]
    L = _side(n, f["rho"])
    basis = np.zeros((1, 3)) if fluid == "salt" else np.array(
        [[0, 0, 0], [0, .5, .5], [.5, 0, .5], [.5, .5, 0]], dtype=np.float64)
    m = int(math.ceil((n / len(basis)) ** (1.0 / 3.0) - 1e-9))
    i = np.arange(m)
    cells = np.stack(np.meshgrid(i, i, i, indexing="ij"), axis=-1).reshape(-1, 1, 3)
    sites = ((cells + basis[None] + 0.25) * (L / m) - L / 2).reshape(-1, 3)
    if len(sites) > n:
        sites = sites[np.sort(rng.choice(len(sites), size=n, replace=False))]
    pos = (sites + rng.uniform(-f["jitter"], f["jitter"], size=sites.shape)).astype(np.float32)
    half, side = np.float32(0.5 * L), np.float32(L)
    pos = np.where(pos >= half, pos - side, np.where(pos < -half, pos + side, pos)).astype(np.float32)
    types = np.zeros(n, np.int32)
    if fluid == "ka":
        types[int(round(0.8 * n)):] = 1
    elif fluid == "salt":
        types[n // 2:] = 1
    types = types[rng.permutation(n)]
    v = rng.standard_normal((n, 3)) * math.sqrt(f["T"] if T is None else T)
    v -= v.mean(axis=0)
    return pos, v.astype(np.float32), types, L


def _pairs(fluid):
    """(sigma, epsilon, cutoff) per type pair and the cutoff method."""
    if fluid == "lj":
        return np.ones((1, 1)), np.ones((1, 1)), 2.5 * np.ones((1, 1)), "sp"
    if fluid == "ka":
        sigma = np.array([[1.0, 0.8], [0.8, 0.88]])
        return sigma, np.array([[1.0, 1.5], [1.5, 0.5]]), 2.5 * sigma, "sf"
    return np.ones((2, 2)), np.ones((2, 2)), 2.5 * np.ones((2, 2)), "sf"


def _tuned_layout(n):
    """(threads per particle, particles per block, list builder) as the autotuner picks them."""
    if n < 2500:
        return 32, 8, 4
    if n <= 8192:
        return 32, 16, 1
    if n < 32768:
        return 8, 64, 3
    if n < 131072:
        return 4, 256, 2
    return (1, 1024, 2) if n < 600000 else (1, 256, 2)


def _system(fluid, start, precision="f32", tuned=0, T=None, layout=None):
    pos, vel, types, L = start
    f = FLUIDS[fluid]
    sigma, eps, rc, method = _pairs(fluid)
    s = srmd.System(pos, types, [L, L, L], vel=vel, ntypes=len(sigma), precision=precision,
                    stream=torch.cuda.current_stream().cuda_stream)
    s.set_skin(SKIN)
    s.set_pairs(sigma, eps, rc, method)
    if fluid == "salt":
        s.set_coulomb_sf([1.0, -1.0], RC_COULOMB)
    if fluid == "lj":
        s.set_integrator_nve(f["dt"])
    else:
        s.set_integrator_nvt(f["dt"], f["T"] if T is None else T, TAU)
    if tuned:
        tp, ppb, builder = _tuned_layout(len(pos))
        s.set_launch(tp, ppb)
        s.set_rebuild_path(0, builder if fluid == "lj" or len(pos) >= 2500 else 1)
    if layout:
        s.set_launch(*layout)
    return s


def _replicas(case, seed):
    """Sizes, temperatures and starts of the replica set (the sizes belong to the case,
    the configurations to the seed)."""
    sizes = np.random.default_rng(2026)
    ns = sizes.integers(case["lo"], case["hi"] + 1, size=case["replicas"])
    ts = sizes.uniform(0.4, 1.0, size=case["replicas"])
    rng = np.random.default_rng(seed)
    return [(int(n), float(t), _start(case["fluid"], int(n), rng, T=float(t))) for n, t in zip(ns, ts)]


def prepare(case, seed):
    kind, fluid = case["kind"], case["fluid"]
    if kind == "batch":
        systems = [_system(fluid, start, T=T, layout=(1, 256)) for _, T, start in _replicas(case, seed)]
        return dict(case=case, systems=systems, batch=srmd.Batch(systems))
    start = _start(fluid, case["n"], np.random.default_rng(seed))
    if kind == "noalloc":
        pos, _, types, L = start
        sigma, eps, rc, method = _pairs(fluid)
        n = case["n"]
        return dict(case=case, cfg=srmd.lj_config(n, [L, L, L], sigma, eps, rc, method, SKIN),
                    pos=torch.from_numpy(pos).cuda(), types=torch.from_numpy(types).cuda(),
                    force=torch.zeros(n, 3, device="cuda"), energy=torch.zeros(2, dtype=torch.float64, device="cuda"),
                    status=torch.zeros(1, dtype=torch.int32, device="cuda"))
    s = _system(fluid, start, case.get("precision", "f32"), case.get("tuned", 0))
    return dict(case=case, system=s, pos=start[0])


def run(state):
    case = state["case"]
    kind = case["kind"]
    if kind == "noalloc":
        srmd.compute_forces_noalloc(state["cfg"], state["pos"].data_ptr(), state["types"].data_ptr(),
                                    state["force"].data_ptr(), state["energy"].data_ptr(), state["status"].data_ptr(),
                                    torch.cuda.current_stream().cuda_stream)
        return state["force"], state["energy"], state["status"]
    if kind == "batch":
        state["batch"].step(case["steps"])
        frames = [s.get_state() for s in state["systems"]]
        return {k: np.concatenate([f[k] for f in frames]) for k in ("pos", "vel", "force", "image")}
    s = state["system"]
    if kind == "forces":
        s.set_state(pos=state["pos"])
        record = s.compute_forces()
        return dict(pe=record["pe"], virial=record["virial"], force=s.get_state()["force"])
    s.step(case["steps"])
    frame = s.get_state()
    out = {k: frame[k] for k in ("pos", "vel", "force", "image")}
    if case["precision"] == "f64pos":
        out["pos64"] = frame["pos64"]
    return out


def work(case):
    fluid, kind = case["fluid"], case["kind"]
    listed_, near = PARTNERS[fluid]
    a, b = OPS[fluid]
    if kind == "batch":
        n, steps = case["replicas"] * (case["lo"] + case["hi"]) / 2, case["steps"]
    else:
        n, steps = case["n"], case.get("steps", 1)
    flops = n * steps * (a * listed_ + b * near)
    if kind in ("noalloc", "forces"):
        return {"bytes": n * (12 + 4 + 12), "flops": flops}
    # a step reads and writes positions and velocities, reads a list entry per listed
    # partner and writes the force
    return {"bytes": n * steps * (48 + 12 + 4 * listed_), "flops": flops}


# ---------------------------------------------------------------- the same in 64 bits

EXACT_PAIRS = 5e9  # candidate pairs of one list build that stay within seconds


def _pair_list(x, L, reach):
    """Ordered pairs (i, j) within reach, by brute force in blocks of rows."""
    n = len(x)
    rows = max(1, int(2e7 // n))
    found = []
    for i0 in range(0, n, rows):
        xi = x[i0:i0 + rows]
        r2 = torch.zeros(len(xi), n, dtype=torch.float32, device=x.device)
        for k in range(3):
            d = (x[None, :, k] - xi[:, None, k]).float()
            d -= L * torch.round(d / L)
            r2 += d * d
        hit = (r2 < reach * reach).nonzero()
        hit[:, 0] += i0
        found.append(hit[hit[:, 0] != hit[:, 1]])
    return torch.cat(found).t().contiguous()


class _Forces64:
    """Forces, potential energy and virial in float64, over a list with a margin."""

    def __init__(self, fluid, types, L):
        dev = types.device
        sigma, eps, rc, method = (torch.as_tensor(v, dtype=torch.float64, device=dev) if not isinstance(v, str) else v
                                  for v in _pairs(fluid))
        s6 = (sigma / rc) ** 6
        self.fluid, self.types, self.L = fluid, types, L
        self.sigma, self.eps, self.rc = sigma, eps, rc
        self.urc = 4 * eps * (s6 * s6 - s6)
        self.frc = 24 * eps * (2 * s6 * s6 - s6) / rc if method == "sf" else torch.zeros_like(rc)
        self.reach = max(float(rc.max()), RC_COULOMB if fluid == "salt" else 0.0)
        self.margin = 0.4
        self.built = None

    def __call__(self, x):
        if self.built is None or float((x - self.built).norm(dim=1).max()) > 0.5 * self.margin:
            self.ij, self.built = _pair_list(x, self.L, self.reach + self.margin), x.clone()
        i, j = self.ij
        d = x[j] - x[i]
        d -= self.L * torch.round(d / self.L)
        r2 = (d * d).sum(1)
        keep = r2 < self.reach * self.reach
        i, j, d, r2 = i[keep], j[keep], d[keep], r2[keep]
        q = self.types[i], self.types[j]
        r = r2.sqrt()
        s6 = (self.sigma[q] ** 2 / r2) ** 3
        inside = (r2 < self.rc[q] ** 2).double()
        fr = inside * (24 * self.eps[q] * (2 * s6 * s6 - s6) / r2 - self.frc[q] / r)
        u = inside * (4 * self.eps[q] * (s6 * s6 - s6) - self.urc[q] + (r - self.rc[q]) * self.frc[q])
        if self.fluid == "salt":
            qq = (1.0 - 2.0 * q[0]) * (1.0 - 2.0 * q[1])
            c = RC_COULOMB
            fr = fr + qq * (1 / r2 - 1 / c ** 2) / r
            u = u + qq * (1 / r - 1 / c + (r - c) / c ** 2)
        F = torch.zeros_like(x).index_add_(0, i, -fr[:, None] * d)
        return F, 0.5 * float(u.sum()), float((fr * r2).sum()) / 6


def _wrap64(x, L):
    return x - L * torch.floor(x / L + 0.5)


def _trajectory64(fluid, start, steps, T):
    dev = "cuda" if torch.cuda.is_available() else "cpu"
    pos, vel, types, L = start
    x = torch.as_tensor(pos, dtype=torch.float64, device=dev)
    v = torch.as_tensor(vel, dtype=torch.float64, device=dev)
    forces = _Forces64(fluid, torch.as_tensor(types, dtype=torch.int64, device=dev), L)
    dt, xi, g = FLUIDS[fluid]["dt"], 0.0, 3 * len(x) - 3
    for _ in range(steps):
        F = forces(x)[0]
        v = (v * (1 - 0.5 * xi * dt) + F * dt) / (1 + 0.5 * xi * dt)
        x = x + v * dt
        if fluid != "lj":
            xi += dt * (float((v * v).sum()) / g / T - 1) / TAU ** 2
    return _wrap64(x, L).cpu(), v.cpu(), F.cpu()


def exact(case, seed):
    kind, fluid = case["kind"], case["fluid"]
    if kind == "batch":
        if case["replicas"] * case["hi"] ** 2 > EXACT_PAIRS / 4:
            return None
        found = [_trajectory64(fluid, start, case["steps"], T) for _, T, start in _replicas(case, seed)]
        pos, vel, force = (torch.cat(v) for v in zip(*found))
        return dict(pos=pos, vel=vel, force=force, image=None)
    if float(case["n"]) ** 2 > EXACT_PAIRS:
        return None
    start = _start(fluid, case["n"], np.random.default_rng(seed))
    if kind == "steps":
        x, v, F = _trajectory64(fluid, start, case["steps"], FLUIDS[fluid]["T"])
        out = dict(pos=x, vel=v, force=F, image=None)
        if case["precision"] == "f64pos":
            out["pos64"] = x
        return out
    dev = "cuda" if torch.cuda.is_available() else "cpu"
    pos, _, types, L = start
    forces = _Forces64(fluid, torch.as_tensor(types, dtype=torch.int64, device=dev), L)
    F, pe, w = forces(torch.as_tensor(pos, dtype=torch.float64, device=dev))
    if kind == "noalloc":
        return F.cpu(), torch.tensor([pe, w], dtype=torch.float64), None
    return dict(pe=pe, virial=w, force=F.cpu())
