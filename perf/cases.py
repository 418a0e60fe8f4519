"""The workloads this library is timed on: whole solves through the public binding.

A pass sets a solve's initial fields, advances it and reads the macroscopic
fields back (``lbm.Solver`` with device or host arrays), or sends a group of
requests through the serving pool (``lbm.Pool``).  The listed cases are the
grids of the benchmark, the paper's shock tubes, the recipes of the tests and
odd sizes between them; ``draw`` gives others of the same ranges.

``exact`` evaluates the scheme itself in float64 with plain torch.
"""
import itertools
import math
import random

import numpy as np
import torch

from paper_1608_06345_amd import lbm

STORES = {"fp64": (lbm.LBM_FP64, 8), "fp32": (lbm.LBM_FP32_DEV, 4),
          "fp16": (lbm.LBM_FP16_SCALED, 2)}
OPEN_X = lbm.LBM_BC(lbm.LBM_BC_ZERO_GRADIENT, lbm.LBM_BC_PERIODIC)
R = 1.196979770393074359  # lattice scale, for the finite-difference time step
PASS_BYTES = 300e9        # no case moves more population bytes than this


def _solve(name, dim, nx, ny, nz, store, steps, gamma=1.4, tau_f=0.65, tau_g=0.65, open_x=False,
           tube=False, fd=False, energy=False, checks=0, host=False):
    """``checks``: how often the totals are read on the way; ``host``: host
    arrays in and out; ``fd``: the finite-difference form (taus in its dt);
    ``energy``: the energy-conserving collision."""
    return dict(name=name, kind="solve", dim=dim, nx=nx, ny=ny, nz=nz, store=store, steps=steps,
                gamma=gamma, tau_f=tau_f, tau_g=tau_g, open_x=open_x, tube=tube, fd=fd,
                energy=energy, checks=checks, host=host)


def listed():
    return [
        # the smallest call: Sod's tube of 200 cells up to the comparison with
        # the exact solution, host arrays as in the README; all launches
        _solve("sod_200x4_fp64_host", 2, 200, 4, 1, "fp64", 48, tau_f=0.8, tau_g=0.8,
               open_x=True, tube=True, host=True),
        # the paper's shock tubes (Sec. V), step 180 in 2D and its first third in 3D
        _solve("tube_1000x16_fp32", 2, 1000, 16, 1, "fp32", 180, tau_f=2 / 3, tau_g=2 / 3,
               open_x=True, tube=True),
        _solve("tube_1000x16x16_fp64", 3, 1000, 16, 16, "fp64", 60, tau_f=2 / 3, tau_g=2 / 3,
               open_x=True, tube=True),
        # an ordinary 2D solve (the 512^2 recipe of the tests) watched by its totals
        _solve("d2q37_512_fp32_watched", 2, 512, 512, 1, "fp32", 80, tau_f=0.7, tau_g=0.8,
               checks=4),
        # 2D at the benchmark's size, double precision
        _solve("d2q37_4096_fp64", 2, 4096, 4096, 1, "fp64", 12, tau_f=0.7, tau_g=0.8),
        # 2D, odd sizes, half storage, the energy-conserving collision
        _solve("d2q37_2047x1531_fp16_energy", 2, 2047, 1531, 1, "fp16", 60, tau_f=0.7, tau_g=0.8,
               energy=True),
        # the headline: D3Q107 at 256^3 in single precision
        _solve("d3q107_256_fp32", 3, 256, 256, 256, "fp32", 10),
        # the 3D recipe of the tests at gamma = 5/3, double precision
        _solve("d3q107_128x64x256_fp64", 3, 128, 64, 256, "fp64", 20, gamma=5 / 3),
        # 3D, odd sizes, half storage
        _solve("d3q107_191x173x187_fp16", 3, 191, 173, 187, "fp16", 24),
        # the finite-difference form: 3D at the benchmark's size, 2D on a ragged grid
        _solve("fd_d3q107_256_fp32", 3, 256, 256, 256, "fp32", 6, tau_f=0.12, tau_g=0.12, fd=True),
        _solve("fd_d2q37_1500x1100_fp64", 2, 1500, 1100, 1, "fp64", 40, tau_f=0.1, tau_g=0.12,
               fd=True),
        # a group of the serving mix (half 2D, a third 3D, the rest tubes)
        # through the pool: admission, 8-step replays, fields to the host
        dict(name="pool_8_fp32", kind="pool", requests=8, mix=5, store="fp32", most=64, ticks=8),
    ]


def _log(rng, lo, hi):
    return math.exp(rng.uniform(math.log(lo), math.log(hi)))


def draw(rng):
    if rng.random() < 0.1:
        return dict(name="", kind="pool", requests=rng.randint(4, 12), mix=rng.randint(0, 10 ** 6),
                    store=rng.choice(["fp32", "fp32", "fp16", "fp64"]), most=64,
                    ticks=rng.choice([4, 8, 16]))
    dim = rng.choice([2, 3])
    fd = rng.random() < 0.3
    tube = rng.random() < 0.25
    store = rng.choice(["fp64", "fp32"] if fd else ["fp64", "fp32", "fp16"])
    cells = _log(rng, 800, 2 ** 24 if dim == 2 else 2 ** 23)
    if tube:  # long and thin
        ny = rng.randint(3, 20)
        nz = rng.randint(3, 20) if dim == 3 else 1
        nx = max(100, min(4000, int(cells / (ny * nz))))
    else:
        side = cells ** (1 / dim)
        nx = max(8, int(side * rng.uniform(0.6, 1.6)))
        ny = max(8, int(side * rng.uniform(0.6, 1.6)))
        nz = max(8, int(cells / (nx * ny))) if dim == 3 else 1
        if rng.random() < 0.4:  # whole cache lines, as grids often are
            nx = -(-nx // 64) * 64
    q = 37 if dim == 2 else 107
    state = 4 * q * STORES[store][1] * nx * ny * nz
    steps = max(4, min(180, int(_log(rng, 2e9, 0.5 * PASS_BYTES) / state)))
    if tube:
        steps = min(steps, nx // 4)  # the waves are still inside
    same = rng.random() < 0.5
    tau = rng.uniform(0.1, 0.14) if fd else rng.uniform(0.64, 0.85)
    return _solve(None, dim, nx, ny, nz, store, steps,
                  gamma=rng.choice([1.4, 1.25, 1.55] + ([5 / 3] if dim == 3 else [2.0])),
                  tau_f=tau, tau_g=tau if same or tube else tau * rng.uniform(0.95, 1.15),
                  open_x=tube or rng.random() < 0.2, tube=tube, fd=fd,
                  energy=not same and rng.random() < 0.5,
                  checks=rng.choice([0, 0, 0, 2]), host=rng.random() < 0.15) | {"name": ""}


def _mix(c):
    """The requests of a pool case (the shape of the serving mix, fewer steps)."""
    rng = random.Random(c["mix"])
    out = []
    for k in range(c["requests"]):
        gamma, steps = round(rng.uniform(1.1, 1.66), 3), rng.randint(c["most"] // 4, c["most"])
        kind = ("2d", "3d", "2d", "tube", "2d", "3d")[k % 6]
        if kind == "2d":
            n = int(_log(rng, 256, 1100))
            s = _solve("", 2, n, n, 1, c["store"], steps, gamma, 0.7, 0.8)
        elif kind == "3d":
            n = int(_log(rng, 40, 100))
            s = _solve("", 3, n, n, n, c["store"], steps, gamma)
        else:
            n = int(_log(rng, 100, 4000))
            s = _solve("", 2, n, 4, 1, c["store"], min(steps, n // 4), gamma, 0.8, 0.8,
                       open_x=True, tube=True)
        out.append(s)
    return out


def _fields(c, seed):
    """Initial rho [cells], u [dim][cells], T [cells] on the GPU (x fastest):
    the smooth recipe (eight seeded low modes a field) or a two-state tube."""
    dim, shape = c["dim"], (c["nx"], c["ny"], c["nz"])
    rng = np.random.default_rng([seed, c["nx"], c["ny"], c["nz"]])
    axes = [torch.arange(n, dtype=torch.float64, device="cuda") / n for n in shape[:dim]]
    n = shape[0] * shape[1] * shape[2]
    if c["tube"]:
        ratio = rng.uniform(2.0, 4.0)
        left = (torch.arange(n, device="cuda") % shape[0]) < shape[0] // 2
        rho = torch.where(left, ratio, 1.0).double()
        return rho, torch.zeros(dim, n, dtype=torch.float64, device="cuda"), torch.ones_like(rho)

    def modes(amp):
        out = torch.zeros(tuple(reversed(shape[:dim])), dtype=torch.float64, device="cuda")
        for _ in range(8):
            arg = float(rng.uniform(0, 2 * math.pi))
            a, k = float(rng.uniform(-1, 1)), rng.integers(-8, 9, dim)
            for d in range(dim):
                view = [1] * dim
                view[dim - 1 - d] = -1
                arg = arg + 2 * math.pi * float(k[d]) * axes[d].reshape(view)
            out += amp * a * torch.cos(arg)
        return out.reshape(-1)

    u = torch.stack([modes(0.02) for _ in range(dim)])
    return 1.0 + modes(0.01), u.contiguous(), 1.0 + modes(0.01)


def _dt(c):
    return (0.25 if c["dim"] == 2 else 0.3) / (3 * R) if c["fd"] else None


def prepare(case, seed):
    c = dict(case)
    if c["kind"] == "pool":
        mix = _mix(c)
        prec, elem = STORES[c["store"]]
        reqs = [lbm.make_request(m["dim"], m["gamma"], m["tau_f"], m["tau_g"], m["nx"], m["ny"],
                                 m["nz"], bc=OPEN_X if m["open_x"] else 0, steps=m["steps"])
                for m in mix]
        budget = sum(lbm.lbm_pool_request_bytes(r, prec) for r in reqs) + (64 << 20)
        fields = []
        for k, m in enumerate(mix):
            rho, u, T = _fields(m, seed * 1000 + k)
            fields.append((rho, u.reshape(-1).contiguous(), T))
        pool = lbm.Pool(budget, 256, prec)
        pool.set_stream(torch.cuda.current_stream())
        return dict(kind="pool", pool=pool, reqs=reqs, fields=fields, ticks=c["ticks"])
    rho, u, T = _fields(c, seed)
    s = lbm.Solver(c["dim"], c["gamma"], c["tau_f"], c["tau_g"], c["nx"], c["ny"], c["nz"],
                   bc=OPEN_X if c["open_x"] else 0, precision=STORES[c["store"]][0], dt=_dt(c),
                   collision=lbm.LBM_COLLISION_ENERGY_CONSERVING if c["energy"]
                   else lbm.LBM_COLLISION_PAPER)
    s.set_stream(torch.cuda.current_stream())
    st = dict(kind="solve", s=s, c=c)
    if c["host"]:
        st["fields"] = tuple(a.cpu().numpy() for a in (rho, u, T))
    else:
        st["fields"] = (rho, u, T)
        st["out"] = dict(rho=torch.empty_like(rho), u=torch.empty_like(u),
                         E=torch.empty_like(rho), T=torch.empty_like(T))
    # a solver takes its collision mode before its first fields
    return st


def run(state):
    if state["kind"] == "pool":
        pool = state["pool"]
        slots = {}
        for k, (r, f) in enumerate(zip(state["reqs"], state["fields"])):
            slots[pool.admit_dev(r, *f)] = k
        out = [None] * len(state["reqs"])
        while slots:
            pool.run(state["ticks"])
            for slot in pool.poll():
                out[slots.pop(slot)] = pool.moments(slot)
                pool.release(slot)
        return out
    s, c = state["s"], state["c"]
    if c["host"]:
        s.init_fields(*state["fields"])
    else:
        lbm.lbm_init_fields_dev(s.h, *state["fields"])
    checks, left = [], c["steps"]
    for k in range(c["checks"]):
        n = left // (c["checks"] - k)
        s.step(n)
        left -= n
        mass, mom, energy = s.totals()
        checks.append([mass, *mom.tolist(), energy])
    s.step(left)
    if c["host"]:
        rho, u, E = s.moments()
        out = dict(rho=rho, u=u, E=E, T=s.temperature())
    else:
        o = state["out"]
        lbm.lbm_moments_dev(s.h, o["rho"], o["u"], o["E"])
        lbm.lbm_temperature_dev(s.h, o["T"])
        out = dict(o)
    out["checks"] = np.array(checks, dtype=np.float64).reshape(-1)
    if not c["checks"]:
        del out["checks"]
    return out


def work(case):
    """Fields in, every step's read and write of the populations, fields out;
    about 20 floating-point operations per population and step."""
    if case["kind"] == "pool":
        w = [work(m) for m in _mix(case)]
        return {k: sum(x[k] for x in w) for k in ("bytes", "flops")}
    n, d = case["nx"] * case["ny"] * case["nz"], case["dim"]
    q = 37 if d == 2 else 107
    state = 2 * q * STORES[case["store"]][1] * n
    return {"bytes": 8 * n * (2 + d) + 2 * state * case["steps"] + 8 * n * (3 + d),
            "flops": 40 * q * n * case["steps"]}


# -- the scheme in float64 ---------------------------------------------------


def _lattice(dim):
    """e [Q][dim], w [Q], r: the group weights and the scale that make the
    discrete Hermite moments up to degree 8 those of the normal weight
    (Newton in extended precision from the printed tables)."""
    reps = ([(0, 0), (1, 0), (1, 1), (2, 0), (2, 1), (3, 0), (3, 1), (3, 3)] if dim == 2 else
            [(0, 0, 0), (1, 0, 0), (1, 1, 0), (1, 1, 1), (2, 0, 0), (2, 1, 1), (2, 2, 0),
             (2, 2, 2), (3, 0, 0), (3, 1, 1)])
    w0 = ([2.03916918e-1, 1.27544846e-1, 4.37537182e-2, 8.13659044e-3, 9.40079914e-3,
           6.95051049e-4, 3.04298494e-5, 2.81093762e-5] if dim == 2 else
          [1.603003550e-1, 2.390868500e-2, 4.169870315e-2, 5.166346780e-3, 1.227117147e-2,
           2.676524495e-3, 9.685223338e-4, 2.170763000e-5, 2.453010230e-4, 1.417071270e-4])
    members = [sorted({tuple(a * b for a, b in zip(p, s)) for p in itertools.permutations(rep)
                       for s in itertools.product((1, -1), repeat=dim)}) for rep in reps]
    ld = np.longdouble
    conds = [a for a in itertools.product(range(0, 9, 2), repeat=dim)
             if sum(a) <= 8 and list(a) == sorted(a, reverse=True)]
    sums = [[ld(sum(math.prod(e[k] ** a[k] for k in range(dim)) for e in m)) for m in members]
            for a in conds]
    want = [ld(math.prod(math.prod(range(1, k, 2)) for k in a)) for a in conds]
    x = np.array(w0 + [1.19697977 ** 2], dtype=ld)
    n = len(x)
    for _ in range(12):
        s = x[-1]
        A = np.zeros((n, n + 1), dtype=ld)
        for c, a in enumerate(conds):
            p = sum(a) // 2
            val = sum(x[g] * sums[c][g] for g in range(n - 1))
            A[c, :n - 1] = [sums[c][g] * s ** p for g in range(n - 1)]
            A[c, n - 1] = p * val * s ** (p - 1) if p else 0
            A[c, n] = want[c] - val * s ** p
        for k in range(n):  # elimination with row pivoting
            p = k + int(np.argmax(np.abs(A[k:, k])))
            A[[k, p]] = A[[p, k]]
            A[k] /= A[k, k]
            for j in range(n):
                if j != k:
                    A[j] -= A[j, k] * A[k]
        x = x + A[:, n]
    e = [v for m in members for v in m]
    w = [float(x[g]) for g, m in enumerate(members) for _ in m]
    return e, w, float(np.sqrt(x[-1]))


def _shift(p, d, axis, open_end):
    """q with q(x) = p(x + d) along one axis (wrapped, or the end value)."""
    if d == 0:
        return p
    if not open_end:
        return torch.roll(p, -d, axis)
    n = p.shape[axis]
    return p.index_select(axis, (torch.arange(n, device=p.device) + d).clamp(0, n - 1))


def _exact_solve(c, seed):
    dim = c["dim"]
    e, w, r = _lattice(dim)
    delta = 2.0 / (c["gamma"] - 1.0) - dim
    delta = 0.0 if abs(delta) < 1e-9 else delta
    shape = (c["nx"], c["ny"], c["nz"])[:dim][::-1]
    rho, u, T = _fields(c, seed)
    rho, u, T = rho.reshape(shape), u.reshape((dim,) + shape), T.reshape(shape)
    dt = _dt(c)
    af, ag = (1 / c["tau_f"], 1 / c["tau_g"]) if dt is None else (dt / c["tau_f"], dt / c["tau_g"])

    def feq(i):
        cc = sum((r * e[i][k]) * u[k] for k in range(dim))
        q, t, U = r * r * sum(k * k for k in e[i]), T - 1.0, UU
        A0 = 1 + (t * (q - dim) - U) / 2 + (3 * U * U + 6 * t * (dim + 2 - q) * U + 3 * t * t * (
            q * q - 2 * (dim + 2) * q + dim * (dim + 2))) / 24
        A1, A2 = 1 - U / 2 + t * (q - dim - 2) / 2, 0.5 - U / 4 + t * (q - dim - 4) / 4
        return w[i] * rho * (A0 + cc * (A1 + cc * (A2 + cc * (1 / 6 + cc / 24))))

    def read():
        s0, sh, s2 = torch.zeros(shape, **o), torch.zeros(shape, **o), torch.zeros(shape, **o)
        sj = [torch.zeros(shape, **o) for _ in range(dim)]
        for i in range(Q):
            s0 += g[i]
            sh += h[i]
            for k in range(dim):
                if e[i][k]:
                    sj[k].add_(g[i], alpha=r * e[i][k])
            s2.add_(g[i], alpha=0.5 * r * r * sum(k * k for k in e[i]))
        uu = torch.stack([s / s0 for s in sj])
        E = (s2 + sh) / s0
        return s0, uu, E, (2 * E - (uu * uu).sum(0)) / (dim + delta), s2

    Q = len(e)
    o = dict(dtype=torch.float64, device="cuda")
    g, h = torch.empty((Q,) + shape, **o), torch.empty((Q,) + shape, **o)
    UU = (u * u).sum(0)
    for i in range(Q):
        g[i] = feq(i)
        h[i] = 0.5 * delta * T * g[i]
    marks, done = {}, 0
    left = c["steps"]
    for k in range(c["checks"]):
        done += left // (c["checks"] - k)
        left -= left // (c["checks"] - k)
        marks[done] = None
    for n in range(1, c["steps"] + 1):
        rho, u, E, T, etr = read()
        UU = (u * u).sum(0)
        kappa = 0.5 * delta * T
        if c["energy"]:
            kappa = kappa + (1 - c["tau_g"] / c["tau_f"]) * (
                0.5 * rho * (UU + dim * T) - etr) / rho
        for i in range(Q):
            F = feq(i)
            for p, target, rate in ((g, F, af), (h, kappa * F, ag)):
                old = p[i].clone()
                new = old + rate * (target - old)
                if dt is None:
                    for k in range(dim):
                        new = _shift(new, -e[i][k], dim - 1 - k, c["open_x"] and k == 0)
                else:
                    for k in range(dim):
                        if e[i][k]:
                            s, ax = (1 if e[i][k] > 0 else -1), dim - 1 - k
                            op = c["open_x"] and k == 0
                            new = new - (dt * r / 6 * abs(e[i][k])) * (
                                _shift(old, -2 * s, ax, op) - 6 * _shift(old, -s, ax, op)
                                + 3 * old + 2 * _shift(old, s, ax, op))
                p[i] = new
        if n in marks:
            a, b, E, _, _ = read()
            marks[n] = [float(a.sum()), *[float((a * b[k]).sum()) for k in range(dim)],
                        float((a * E).sum())]
    rho, u, E, T, _ = read()
    out = dict(rho=rho.reshape(-1), u=u.reshape(dim, -1), E=E.reshape(-1), T=T.reshape(-1))
    if c["checks"]:
        out["checks"] = np.array([marks[k] for k in sorted(marks)]).reshape(-1)
    return out


def _exact_seconds(c):
    q = 37 if c["dim"] == 2 else 107
    n = c["nx"] * c["ny"] * c["nz"]
    return c["steps"] * q * 50 * (1e-5 + n * 24 / 4e12) * (2 if c["fd"] else 1)


def exact(case, seed):
    parts = _mix(case) if case["kind"] == "pool" else [case]
    if sum(_exact_seconds(m) for m in parts) > 18:
        return None
    if case["kind"] == "solve":
        return _exact_solve(case, seed)
    return [tuple(_exact_solve(m, seed * 1000 + k)[f] for f in ("rho", "u", "E"))
            for k, m in enumerate(parts)]
