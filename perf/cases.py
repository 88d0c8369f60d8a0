"""Performance cases of the library: what its users run, at the sizes they run it.

A pass is one stretch of a simulation as a program drives it through the binding: ``step(k)``,
then the masses (with the positions where the program takes a snapshot it can resume from) and
the conservation statistics read back to the host.  Two cases differ: a whole life of a small
simulation (create, step, read, close), and a mix of independent simulations served through the
pool.  The workloads are those of ``workloads.py`` at their own densities, time steps and
diffusivities; positions, masses and the random-walk key come from the seed.

``exact`` repeats a pass in plain torch in FP64.  In the FP32 modes the positions are FP32 state by
definition (rounded at create, walked in FP32), so it keeps them in FP32 and does all the rest in FP64.
"""
import math
from dataclasses import replace

import numpy as np
import torch

from paper_2204_03756_amd import mtpt, serve, workloads as W

LARGEST_PARTICLE_STEPS = 3.2e9          # particles times steps of the largest listed pass
EXACT_PARTICLE_STEPS = 6e8              # the FP64 repeat of more than this takes too long


def listed():
    return [
        # a program that reads the state after every step of a tiny simulation (an animation, a
        # coupling to another code): launches and latency are all it pays
        {"name": "walk2d_1e3_every_step", "work": "rw2d", "n": 1000, "steps": 1, "precision": "fp32w", "read": "state"},
        # the pure mass-transfer workload as configured: 1e4 particles, 50 steps, FP64
        {"name": "transfer2d_1e4_f64", "work": "plain2d", "n": 10_000, "steps": 50, "precision": "fp64",
         "read": "masses"},
        # the same physics on a larger, ragged set of particles with FP32 weights
        {"name": "transfer2d_3e5_f32w", "work": "plain2d", "n": 300_007, "steps": 50, "precision": "fp32w",
         "read": "masses"},
        # the 2-d random-walk workload as configured
        {"name": "walk2d_4e6_f32w", "work": "rw2d", "n": 4_000_000, "steps": 100, "precision": "fp32w",
         "read": "masses"},
        # a ragged 2-d run in full precision, with a snapshot to resume from
        {"name": "walk2d_1e6_f64", "work": "rw2d", "n": 1_000_003, "steps": 50, "precision": "fp64", "read": "state"},
        # anisotropic dispersion (a rotated tensor), 2-d
        {"name": "tensor2d_5e5_f32w", "work": "aniso2d", "n": 500_009, "steps": 50, "precision": "fp32w",
         "read": "masses"},
        # the 3-d random-walk workload as configured: about 28 neighbours per particle
        {"name": "walk3d_2e6_f32w", "work": "rw3d", "n": 2_000_000, "steps": 100, "precision": "fp32w",
         "read": "masses"},
        # a small 3-d run in the all-FP32 compensated mode, with a snapshot
        {"name": "walk3d_1e5_kahan", "work": "rw3d", "n": 100_003, "steps": 60, "precision": "kahan", "read": "state"},
        # the reacting benchmark workload at its full size: 3.2e7 particles of three species
        {"name": "react3d_3e7_f32w", "work": "react3d", "n": 32_000_000, "steps": 100, "precision": "fp32w",
         "read": "masses"},
        # a ragged reacting run in full precision
        {"name": "react3d_1e6_f64", "work": "react3d", "n": 1_000_001, "steps": 50, "precision": "fp64",
         "read": "masses"},
        # one member of a parameter study: a simulation created, run, read and closed
        {"name": "life3d_5e4_f32w", "work": "rw3d", "n": 50_021, "steps": 20, "precision": "fp32w", "read": "state",
         "life": True},
        # the serving mix, in a closed loop: independent 2-d and 3-d simulations of 1e4 to 1e6 particles
        {"name": "serve_16", "work": "serve", "requests": 16, "mix": 20220404, "n_min": 10_000, "n_max": 1_000_000,
         "precision": "kahan"},
    ]


# particles of a drawn case: from a thousand to the size its workload is configured at (the
# static workload, configured at 1e4, also on larger sets)
_DRAW_N = {"plain2d": 1_000_000, "rw2d": 4_000_000, "adv2d": 4_000_000, "aniso2d": 4_000_000, "rw3d": 2_000_000,
           "react3d": 32_000_000}


def draw(rng):
    if rng.random() < 0.15:
        n_max = int(10 ** rng.uniform(4.5, 6.0))
        return {"work": "serve", "requests": rng.randint(2, 16), "mix": rng.randint(1, 10_000_000), "n_min": 10_000,
                "n_max": n_max, "precision": rng.choice(["kahan", "kahan", "fp32w", "fp64"])}
    work = rng.choice(sorted(_DRAW_N) + ["react3d", "rw3d", "rw2d"])
    n = int(10 ** rng.uniform(3.0, math.log10(_DRAW_N[work])))
    steps = int(round(10 ** rng.uniform(0.0, 2.0)))
    # FP64 steps take up to about twice the FP32 ones
    precision = rng.choice(["fp32w", "fp32w", "fp64", "kahan"])
    most = LARGEST_PARTICLE_STEPS / (2.5 if precision == "fp64" else 1.2)
    steps = max(1, min(steps, int(most / n)))
    case = {"work": work, "n": n, "steps": steps, "precision": precision,
            "read": rng.choice(["masses", "masses", "state"]) if n < 3_000_000 else "masses"}
    if n < 300_000 and rng.random() < 0.2:
        case["life"] = True
    return case


# ------------------------------------------------------------------ inputs
def _params(work, n, precision, key):
    """The workload's parameters at n particles (its density), as workloads.py sets them."""
    if work == "plain2d":
        dim, L, d_rw, d_mt, dt = 2, 100.0 * math.sqrt(n / 1e4), 0.0, 1.0, 0.1
    elif work in ("rw2d", "adv2d", "aniso2d"):
        dim, L, d_rw, d_mt, dt = 2, 2000.0 * math.sqrt(n / 4e6), 0.5, 0.5, 0.1
    elif work == "rw3d":
        dim, L, d_rw, d_mt, dt = 3, 126.0 * (n / 2e6) ** (1.0 / 3.0), 1.0, 1.0, 0.1
    elif work == "react3d":
        dim, L, d_rw, d_mt, dt = 3, 318.0 * (n / 3.2e7) ** (1.0 / 3.0), 0.3, 0.7, 0.05
    else:
        raise ValueError(work)
    p = W.Params(dim=dim, n=n, lo=[0.0] * 3, hi=[L] * dim + [0.0] * (3 - dim), d_rw=d_rw, d_mt=d_mt, dt=dt, beta=0.5,
                 seed=key, precision=W.PRECISIONS[precision])
    if work == "adv2d":
        p = replace(p, vel=[1.0, 0.5, 0.0])
    if work == "aniso2d":
        p = replace(p, disp=W.rotated_tensor([2.0, 0.5], [math.pi / 6]))
    if work == "react3d":
        p = replace(p, n_species=3, k_react=1.0)
    return p


def _positions(p, rng):
    x = rng.random((p.n, p.dim))
    x *= np.asarray(p.hi[:p.dim])
    return x


def _masses(work, p, x):
    L = p.hi[0]
    if work in ("plain2d", "serve"):
        return (x[:, 0] < L / 2).astype(np.float64)[None, :]
    if work == "react3d":
        m = np.zeros((3, p.n))
        m[0] = x[:, 0] < L / 2
        m[1] = 1.0 - m[0]
        return m
    c = L / 2
    r2 = ((x - c) ** 2).sum(axis=1)
    if work == "rw3d":                       # a point-like source on the particles nearest the centre
        src = max(1, min(1000, p.n // 2000))
        m = np.zeros((1, p.n))
        m[0, np.argpartition(r2, src - 1)[:src]] = 1e-3
        return m
    sigma = 50.0 * L / 2000.0
    return np.exp(-r2 / (2.0 * sigma * sigma))[None, :]


def _inputs(case, seed):
    """[(params, positions, masses, steps)] of the pass: one simulation, or the mix of a pool."""
    rng = np.random.Generator(np.random.SFC64(seed))
    key = 0x4D54505400000000 + seed % (1 << 24)
    if case["work"] != "serve":
        p = _params(case["work"], case["n"], case["precision"], key)
        x = _positions(p, rng)
        return [(p, x, _masses(case["work"], p, x), case["steps"])]
    sims = []
    for r in _mix(case):
        p = replace(r.params, seed=key + (r.rid << 24))
        x = _positions(p, rng)
        sims.append((p, x, _masses("serve", p, x), r.steps))
    return sims


def _mix(case):
    return [W.request(k, base_seed=case["mix"], n_min=case["n_min"], n_max=case["n_max"],
                      precision=W.PRECISIONS[case["precision"]]) for k in range(case["requests"])]


# ------------------------------------------------------------------- a pass
_ALLOCATOR = []


def _allocator():
    if not _ALLOCATOR:
        _ALLOCATOR.append(mtpt.TorchAllocator("cuda:0"))
    return _ALLOCATOR[0]


def prepare(case, seed):
    sims = _inputs(case, seed)
    if case["work"] == "serve":
        requests = [W.Request(k, 0.0, p, x, m, steps) for k, (p, x, m, steps) in enumerate(sims)]
        return {"case": case, "requests": requests, "pool": serve.PoolBackend(allocator=_allocator())}
    p, x, m, _ = sims[0]
    if case.get("life"):
        return {"case": case, "params": p, "x0": x, "m0": m}
    return {"case": case, "sim": mtpt.Sim(p, x, m, allocator=_allocator())}


def run(state):
    case = state["case"]
    if case["work"] == "serve":
        rep = serve.serve(state["pool"], state["requests"])
        return [{"masses": rep.outcomes[r.rid].masses, "pairs": rep.outcomes[r.rid].pairs_total}
                for r in state["requests"]]
    if case.get("life"):
        with mtpt.Sim(state["params"], state["x0"], state["m0"], allocator=_allocator()) as sim:
            return _advance(sim, case)
    return _advance(state["sim"], case)


def _advance(sim, case):
    sim.step(case["steps"])
    out = {"masses": sim.masses()}
    if case["read"] == "state":
        out["positions"] = sim.positions()
    st = sim.stats()
    out["pairs"] = st["pairs_last"]
    out["mass_total"] = np.array(st["mass_total"][:sim.ns])
    return out


def work(case):
    """Every step reads and writes the particles' state once (a static simulation's positions are only
    read) and evaluates each ordered pair within psi once; what is read back is written once more."""
    if case["work"] == "serve":
        sims = [(r.params, r.steps) for r in _mix(case)]
    else:
        sims = [(_params(case["work"], case["n"], case["precision"], 0), case["steps"])]
    total_bytes = flops = 0.0
    for p, steps in sims:
        pos = p.dim * (8 if p.precision == W.FP64 else 4)
        mass = p.n_species * (4 if p.precision == W.FP32_KAHAN else 8)
        moving = p.d_rw > 0
        volume = math.pi * p.psi_eff ** 2 if p.dim == 2 else 4.0 / 3.0 * math.pi * p.psi_eff ** 3
        volume *= math.sqrt(np.linalg.det(np.array(p.disp).reshape(3, 3))) if any(p.disp) else 1.0
        pairs = max(0.0, p.n / p.volume * volume - 1.0)
        total_bytes += steps * p.n * (2 * (pos + mass) if moving else pos + 2 * mass)
        total_bytes += p.n * 8.0 * (p.n_species + (p.dim if case.get("read") == "state" else 0))
        # r^2, scale and exponential, row sum, weight, three operations a species; the walk's normals
        flops += steps * p.n * (pairs * (3 * p.dim - 1 + 6 + 3 * p.n_species) + (40 * p.dim if moving else 0))
    return {"bytes": total_bytes, "flops": flops}


# ------------------------------------------------- the same pass in 64 bits
def exact(case, seed):
    if case["work"] == "serve":
        total = sum(r.params.n * r.steps for r in _mix(case))
    else:
        total = case["n"] * case["steps"]
    if total > EXACT_PARTICLE_STEPS:
        return None
    out = []
    for p, x, m, steps in _inputs(case, seed):
        masses, positions, pairs, pairs_total = _simulate(p, x, m, steps)
        one = {"masses": masses.cpu().numpy()}
        if case["work"] == "serve":
            one["pairs"] = pairs_total
        else:
            if case["read"] == "state":
                one["positions"] = positions.double().cpu().numpy()
            one["pairs"] = pairs
            one["mass_total"] = masses.sum(dim=1).cpu().numpy()
        out.append(one)
    return out if case["work"] == "serve" else out[0]


def _philox(pid, call, step, key):
    """Philox4x32-10 of the counters (pid, call, step): four words per particle, as int64."""
    mask = 0xFFFFFFFF
    c = [pid, torch.full_like(pid, call), torch.full_like(pid, step & mask), torch.full_like(pid, step >> 32)]
    k0, k1 = key & mask, (key >> 32) & mask
    for _ in range(10):
        p0, p1 = c[0] * 0xD2511F53, c[2] * 0xCD9E8D57        # modulo 2^64
        c = [((p1 >> 32) & mask) ^ c[1] ^ k0, p1 & mask, ((p0 >> 32) & mask) ^ c[3] ^ k1, p0 & mask]
        k0, k1 = (k0 + 0x9E3779B9) & mask, (k1 + 0xBB67AE85) & mask
    return c


def _normals(n, dim, step, key, device):
    pid = torch.arange(n, dtype=torch.int64, device=device)
    z = []
    for call in range((dim + 1) // 2):
        w = _philox(pid, call, step, key)
        u1 = (2 * ((w[1] << 20) | (w[0] >> 12)) + 1).double() * 2.0 ** -53
        u2 = (2 * ((w[3] << 20) | (w[2] >> 12)) + 1).double() * 2.0 ** -53
        r = torch.sqrt(-2.0 * torch.log(u1))
        z += [r * torch.cos(2.0 * math.pi * u2), r * torch.sin(2.0 * math.pi * u2)]
    return torch.stack(z[:dim], dim=1)


def _pairs(x, lo, hi, reach, psi2, minv):
    """Ordered pairs (i, j), i != j, with q(x_i, x_j) <= psi2, and q: cells of side >= reach, one row
    of three cells at a time."""
    n, dim = x.shape
    nc = [max(1, min(int((hi[k] - lo[k]) / (reach[k] * (1 + 1e-6))), 1 << 20)) for k in range(dim)]
    while math.prod(nc) > max(64, 4 * n):
        nc = [max(1, c - max(1, c // 8)) for c in nc]
    cell = [((x[:, k] - lo[k]) * (nc[k] / (hi[k] - lo[k]))).long().clamp_(0, nc[k] - 1) for k in range(dim)]
    lin = cell[dim - 1]
    for k in range(dim - 2, -1, -1):
        lin = lin * nc[k] + cell[k]
    order = torch.argsort(lin)
    start = torch.zeros(math.prod(nc) + 1, dtype=torch.int64, device=x.device)
    start[1:] = torch.cumsum(torch.bincount(lin, minlength=math.prod(nc)), 0)
    first, last = (cell[0] - 1).clamp_(min=0), (cell[0] + 1).clamp_(max=nc[0] - 1)
    found = []
    for dz in (-1, 0, 1) if dim == 3 else (0,):
        for dy in (-1, 0, 1):
            cy = cell[1] + dy
            ok = (cy >= 0) & (cy < nc[1])
            row = cy
            if dim == 3:
                cz = cell[2] + dz
                ok &= (cz >= 0) & (cz < nc[2])
                row = cz * nc[1] + cy
            row = torch.where(ok, row, torch.zeros_like(row)) * nc[0]
            b = start[row + first]
            count = torch.where(ok, start[row + last + 1] - b, torch.zeros_like(b))
            i = torch.repeat_interleave(torch.arange(n, device=x.device), count)
            ends = torch.cumsum(count, 0)
            j = order[torch.arange(i.numel(), device=x.device) - (ends - count)[i] + b[i]]
            d = x[j] - x[i]
            if minv is not None:
                d = d @ minv.T
            d = d * d
            q = d[:, 0] + d[:, 1]
            if dim == 3:
                q = q + d[:, 2]
            keep = (q <= psi2) & (i != j)
            found.append((i[keep], j[keep], q[keep]))
    return [torch.cat(v) for v in zip(*found)]


def _simulate(p, x0, m0, steps):
    device = torch.device("cuda" if torch.cuda.is_available() else "cpu")
    state = torch.float64 if p.precision == W.FP64 else torch.float32
    x = torch.from_numpy(x0).to(device).to(state)
    m = torch.from_numpy(m0).to(device)
    psi, dim = p.psi_eff, p.dim
    chol = minv = None
    reach = [psi] * dim
    if any(p.disp):
        t = torch.tensor(p.disp, dtype=torch.float64).reshape(3, 3)[:dim, :dim]
        chol = torch.linalg.cholesky(t)
        minv = torch.linalg.inv(chol).to(device)
        reach = [psi * math.sqrt(float(t[k, k])) for k in range(dim)]
        chol = chol.to(device)
    moving = p.d_rw > 0 or any(p.vel[:dim])
    lo = torch.tensor(p.lo[:dim], dtype=torch.float64, device=device).to(state)
    hi = torch.tensor(p.hi[:dim], dtype=torch.float64, device=device).to(state)
    drift = torch.tensor(p.vel[:dim], dtype=torch.float64, device=device) * p.dt
    to_c = p.n / p.volume
    pairs = pairs_total = 0
    for step in range(steps):
        if moving:
            z = _normals(p.n, dim, p.start_step + step, p.seed, device)
            if chol is not None:
                z = z @ chol.T
            x = x + (z * math.sqrt(2.0 * p.d_rw * p.dt) + drift).to(state)
            while True:
                below, above = x < lo, x > hi
                if not bool((below | above).any()):
                    break
                x = torch.where(below, 2.0 * lo - x, torch.where(above, 2.0 * hi - x, x))
        if moving or step == 0:
            i, j, q = _pairs(x.double(), p.lo, p.hi, reach, psi * psi, minv)
            k = torch.exp(-p.beta / (4.0 * p.d_mt * p.dt) * q)
            s = torch.ones(p.n, dtype=torch.float64, device=device).index_add_(0, i, k)
            w = 2.0 * k / (s[i] + s[j])
            pairs = int(i.numel())
        m = torch.stack([c + p.beta * torch.zeros_like(c).index_add_(0, i, w * (c[j] - c[i])) for c in m])
        if p.n_species == 3 and p.k_react > 0:
            a, b = torch.maximum(m[0], m[1]) * to_c, torch.minimum(m[0], m[1]) * to_c
            d = a - b
            left = torch.where(d > 0, a * d / (d - b * torch.expm1(-p.k_react * d * p.dt)).clamp_min(1e-300),
                               a / (1.0 + p.k_react * a * p.dt))
            gone = (a - left) / to_c
            m = torch.stack([m[0] - gone, m[1] - gone, m[2] + gone])
        pairs_total += pairs
    return m, x, pairs, pairs_total
