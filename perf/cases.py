"""The work a program has this library do, as cases that can be timed and checked.

A pass advances a lattice (or an ensemble) by a number of steps and reads its
fields, takes one porosity gradient, or restarts from saved populations: through
the package's public calls, on inputs made from a seed.  ``exact`` states what a
pass returns, by plain torch arithmetic in 64 bits that shares no code with the
package.

Families ("kind"):
  box        fully periodic D3Q19 box, Taylor-Green flow
  channel    D3Q19 channel of solid spheres between walls, driven by a body force
  plane      D2Q9 channel between two walls, driven by a body force
  cavity     D2Q9 lid-driven cavity, moving top wall
  ensemble   many periodic D3Q19 boxes of uneven size in one batch
  adjoint    dJ/dd of the porous D3Q19 channel through autograd
  restart    populations in, one step, populations, totals and fields out
"""
from __future__ import annotations

import functools
import math

import numpy as np
import torch

import paper_2307_11752_amd as lbm
from paper_2307_11752_amd import adjoint, workloads

BYTES = {"f64": 8, "f32": 4, "f16": 2, "bf16": 2}
DEVICE = "cuda"

# Floating-point operations of one cell's BGK collision (moments, equilibrium by
# opposite pairs, relaxation), and of the Guo source where a force acts.
FLOPS = {9: 90, 19: 200}
FORCE_FLOPS = {9: 60, 19: 140}
# Adjoint of one porous collision (state, moments of the adjoint, update).
ADJOINT_FLOPS = 400


def listed():
    return [
        # A program that looks at the flow after every step on a small lattice:
        # launches and calls, not bandwidth.  Direct launches, FP32.
        {"name": "box32_step1", "kind": "box", "nx": 32, "ny": 32, "nz": 32, "storage": "f32",
         "shifted": False, "graph": 0, "steps": 1},
        # The 64 x 64 lid-driven cavity in FP64, 100 steps between looks, replayed
        # as a 100-step graph as the benchmark does.
        {"name": "cavity64_f64", "kind": "cavity", "nx": 64, "ny": 64, "nz": 1, "storage": "f64",
         "shifted": False, "graph": 100, "steps": 100},
        # A 2-D channel flow of the size of the guide's backward-facing step
        # example (about 109,000 nodes), weight-shifted FP32, direct launches.
        {"name": "plane730_f32", "kind": "plane", "nx": 730, "ny": 150, "nz": 1, "storage": "f32",
         "shifted": True, "graph": 0, "steps": 50},
        # Odd edges on every axis, as a box sized by physics and not by lanes has.
        {"name": "box_odd_f32", "kind": "box", "nx": 101, "ny": 77, "nz": 53, "storage": "f32",
         "shifted": False, "graph": 0, "steps": 50},
        # A medium cube in BF16 storage, replayed as graphs.
        {"name": "box96_bf16", "kind": "box", "nx": 96, "ny": 96, "nz": 96, "storage": "bf16",
         "shifted": True, "graph": 50, "steps": 50},
        # The headline flow: Taylor-Green 256^3, a 20-step window, FP32 and FP16.
        {"name": "tgv256_f32", "kind": "box", "nx": 256, "ny": 256, "nz": 256, "storage": "f32",
         "shifted": False, "graph": 0, "steps": 20},
        {"name": "tgv256_f16", "kind": "box", "nx": 256, "ny": 256, "nz": 256, "storage": "f16",
         "shifted": True, "graph": 0, "steps": 20},
        # The sphere-filled channel with walls and forcing, FP32 and FP16.
        {"name": "channel512_f32", "kind": "channel", "nx": 512, "ny": 128, "nz": 128,
         "storage": "f32", "shifted": True, "graph": 0, "steps": 20},
        {"name": "channel512_f16", "kind": "channel", "nx": 512, "ny": 128, "nz": 128,
         "storage": "f16", "shifted": True, "graph": 0, "steps": 20},
        # The 256-lattice ensemble, autotuned, 100-step graphs.
        {"name": "ensemble256_f32", "kind": "ensemble", "count": 256, "lmin": 16, "lmax": 96,
         "boxes": 1107, "storage": "f32", "shifted": False, "graph": 100, "steps": 100},
        # The porosity gradient of the 128 x 64 x 64 channel over 500 steps,
        # a checkpoint every 50.
        {"name": "adjoint128", "kind": "adjoint", "nx": 128, "ny": 64, "nz": 64, "steps": 500,
         "every": 50},
        # Restart from a checkpoint: FP64 populations in, a step, everything out
        # (populations, totals, host fields), in a channel of spheres.
        {"name": "restart128_f64", "kind": "restart", "nx": 128, "ny": 96, "nz": 80,
         "storage": "f64", "shifted": False, "graph": 0, "steps": 1},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


# A drawn lattice moves at most what the 20-step 256^3 FP32 window moves.
_MOST_BYTES = 256 ** 3 * 20 * 2 * 19 * 4


def _steps(rng, q, cells, storage, most=100):
    hi = int(_MOST_BYTES // (cells * 2 * q * BYTES[storage]))
    return _log_int(rng, 1, max(1, min(most, hi)))


def draw(rng):
    kind = rng.choice(["box", "box", "box", "channel", "channel", "plane", "cavity", "ensemble",
                       "adjoint", "restart"])
    if kind == "adjoint":
        every = _log_int(rng, 1, 40)
        c = {"kind": kind, "nx": _log_int(rng, 12, 128), "ny": _log_int(rng, 8, 64),
             "nz": _log_int(rng, 8, 64), "every": every}
        c["steps"] = every + _log_int(rng, 1, 300)
        return c
    storage = rng.choice(["f32", "f32", "f16", "bf16", "f64"])
    c = {"kind": kind, "storage": storage,
         # 16-bit storage is always used shifted; the others either way
         "shifted": storage in ("f16", "bf16") or rng.random() < 0.5}
    if kind == "ensemble":
        lmin = _log_int(rng, 8, 32)
        c.update(count=_log_int(rng, 2, 128), lmin=lmin, lmax=min(96, lmin * rng.randint(2, 4)),
                 boxes=rng.randrange(1 << 20))
        cells = c["count"] * (0.5 * (c["lmin"] + c["lmax"])) ** 3
        c["steps"] = _steps(rng, 19, cells, storage)
        c["graph"] = rng.choice([0, 2 * _log_int(rng, 1, 50)])
        return c
    if kind == "restart":
        c.update(nx=_log_int(rng, 16, 128), ny=_log_int(rng, 8, 96), nz=_log_int(rng, 8, 80),
                 storage="f64", steps=rng.randint(0, 3), graph=0)
        return c
    if kind in ("plane", "cavity"):
        hi = 2048 if kind == "plane" else 512
        c.update(nx=_log_int(rng, 24, hi), ny=_log_int(rng, 16, hi // 2), nz=1)
        if kind == "cavity":
            c["ny"] = c["nx"]
    elif kind == "channel":
        c.update(nx=_log_int(rng, 32, 512), ny=_log_int(rng, 16, 128), nz=_log_int(rng, 16, 128))
    else:
        c.update(nx=_log_int(rng, 16, 256), ny=_log_int(rng, 16, 256), nz=_log_int(rng, 16, 256))
        if rng.random() < 0.3:  # powers of two are common
            for a in ("nx", "ny", "nz"):
                c[a] = 2 ** round(math.log2(c[a]))
    q = 9 if kind in ("plane", "cavity") else 19
    c["steps"] = _steps(rng, q, c["nx"] * c["ny"] * c["nz"], storage)
    c["graph"] = rng.choice([0, 2 * _log_int(rng, 1, 50)])
    return c


# ---------------------------------------------------------------------------
# Inputs
# ---------------------------------------------------------------------------
TAU = {"box": 0.8, "channel": 0.7, "plane": 0.9, "cavity": 0.6, "adjoint": 0.7, "restart": 0.7}


def _flow(shape, seed):
    """Taylor-Green velocity of one period per edge, its amplitude and phases
    from the seed: (3, nz, ny, nx) float64 on the GPU."""
    nx, ny, nz = shape
    r = np.random.default_rng(seed)
    u0, ph = r.uniform(0.02, 0.06), r.uniform(0, 2 * math.pi, 3)
    kx, ky, kz = (2 * math.pi / n for n in shape)

    def axis(n, k, p):
        return torch.arange(n, dtype=torch.float64, device=DEVICE) * k + p

    x = axis(nx, kx, ph[0])[None, None, :]
    y = axis(ny, ky, ph[1])[None, :, None]
    z = axis(nz, kz, ph[2])[:, None, None]
    u = torch.zeros((3, nz, ny, nx), dtype=torch.float64, device=DEVICE)
    u[0] = u0 * torch.sin(x) * torch.cos(y) * torch.cos(z)
    u[1] = -u0 * (kx / ky) * torch.cos(x) * torch.sin(y) * torch.cos(z)
    u[:2] *= min(1.0, 0.08 / float(u.abs().max()))
    return u


def _problem(case, seed):
    """(q, material (nz, ny, nx), periodic axes, initial velocity or None, force, wall velocity)."""
    kind, shape = case["kind"], (case["nx"], case["ny"], case["nz"])
    nx, ny, nz = shape
    r = np.random.default_rng(seed)
    if kind == "box":
        return 19, np.ones((nz, ny, nx), np.uint8), 7, _flow(shape, seed), (0, 0, 0), (0, 0, 0)
    if kind in ("channel", "restart"):
        radius = min(10.0, 0.25 * min(shape))
        wl = workloads.channel_spheres(nx, ny, nz, seed=seed, rmin=0.4 * radius, rmax=radius)
        return 19, wl.material, wl.periodic, _flow(shape, seed), (1e-6, 0, 0), (0, 0, 0)
    if kind == "plane":
        mat = np.ones((1, ny, nx), np.uint8)
        mat[0, 0], mat[0, -1] = 2, 2
        return 9, mat, 1, _flow(shape, seed), (float(r.uniform(0.5e-5, 2e-5)), 0, 0), (0, 0, 0)
    wl = workloads.cavity2d(nx)
    return 9, wl.material, 0, None, (0, 0, 0), (float(r.uniform(0.03, 0.07)), 0, 0)


@functools.cache
def _worker():
    """The program's own stream: replaying graphs needs one."""
    return torch.cuda.Stream()


def _lattice(case, problem):
    q, mat, periodic, u, g, uw = problem
    stream = _worker() if case["graph"] else None
    lat = lbm.Lattice(lbm.D2Q9 if q == 9 else lbm.D3Q19, (case["nx"], case["ny"], case["nz"]),
                      TAU[case["kind"]], storage=case["storage"], shifted=case["shifted"],
                      stream=stream)
    lat.set_geometry(mat, periodic)
    lat.set_body_force(g)
    lat.set_wall_velocity(uw)
    if case["graph"]:
        lat.set_graph_steps(case["graph"])
    lat.init_equilibrium(None, u)
    return lat


def _ensemble(case, seed):
    """Shapes (from the case's own seed) and relaxation times of the members."""
    shapes, _, _ = workloads.tgv_ensemble(case["count"], seed=case["boxes"], lmin=case["lmin"],
                                          lmax=case["lmax"])
    return shapes, np.random.default_rng(seed).uniform(0.55, 1.0, len(shapes))


def _porous(case, seed):
    mat, por = workloads.porous_channel(case["nx"], case["ny"], case["nz"], seed=seed)
    g = (float(np.random.default_rng(seed).uniform(0.5e-5, 2e-5)), 0.0, 0.0)
    return mat, por.astype(np.float32), g


def prepare(case, seed):
    torch.cuda.set_device(0)
    kind = case["kind"]
    if kind == "ensemble":
        shapes, tau = _ensemble(case, seed)
        fields = [_flow(s, seed + k) for k, s in enumerate(shapes)]
        batch = lbm.Batch(lbm.D3Q19, shapes, tau, storage=case["storage"],
                          shifted=case["shifted"], stream=_worker())

        def init():
            for m, u in zip(batch, fields):
                m.init_equilibrium(None, u)

        init()
        batch.autotune()  # advances the members
        init()
        if case["graph"]:
            batch.set_graph_steps(case["graph"])
        return {"case": case, "batch": batch}
    if kind == "adjoint":
        mat, por, g = _porous(case, seed)
        channel = adjoint.PorousChannel(mat, 1, TAU[kind], g, case["steps"], case["every"])
        return {"case": case, "channel": channel,
                "porosity": torch.from_numpy(por).to(DEVICE).requires_grad_()}
    problem = _problem(case, seed)
    state = {"case": case, "lat": _lattice(case, problem)}
    if kind == "restart":
        state["saved"] = _saved(problem, seed)
    return state


def _saved(problem, seed):
    """The populations of a checkpoint: a sheared, slightly uneven equilibrium plus a
    non-equilibrium part; (q, nz, ny, nx) float64, 0 off the fluid."""
    q, mat, _, u, _, _ = problem
    f = _equilibrium(q, u.reshape(3, -1)).reshape(q, *mat.shape)
    gen = torch.Generator(device=DEVICE).manual_seed(seed)
    f *= 1 + 1e-3 * torch.rand(f.shape, dtype=torch.float64, device=DEVICE, generator=gen)
    return f * torch.from_numpy(mat == 1).to(DEVICE)


def run(state):
    case = state["case"]
    kind = case["kind"]
    if kind == "ensemble":
        batch = state["batch"]
        batch.step(case["steps"])
        fields = [m.moments_device() for m in batch]
        return {"rho": torch.cat([r.reshape(-1) for r, _ in fields]),
                "u": torch.cat([u.reshape(3, -1) for _, u in fields], dim=1)}
    if kind == "adjoint":
        d = state["porosity"]
        d.grad = None
        objective = adjoint.porous_objective(d, state["channel"])
        objective.backward()
        return {"objective": objective.detach(), "grad": d.grad}
    lat = state["lat"]
    if kind == "restart":
        lat.set_populations(state["saved"])
        lat.step(case["steps"])
        mass, momentum, stats = lat.totals()
        rho, u = lat.moments()
        return {"f": lat.get_populations(), "mass": mass, "momentum": momentum, "stats": stats,
                "rho": rho, "u": u}
    lat.step(case["steps"])
    rho, u = lat.moments_device()
    return {"rho": rho, "u": u}


def work(case):
    """What a pass cannot do without: the state read once and written once, the
    fields (or gradient) written, and the collisions' arithmetic."""
    kind = case["kind"]
    if kind == "ensemble":
        cells = sum(a * b * c for a, b, c in _ensemble(case, 0)[0])
        return {"bytes": cells * (2 * 19 * BYTES[case["storage"]] + 16),
                "flops": cells * case["steps"] * FLOPS[19]}
    cells = case["nx"] * case["ny"] * case["nz"]
    if kind == "adjoint":
        # porosity in, gradient out; a forward and a reverse sweep
        return {"bytes": cells * 8,
                "flops": cells * case["steps"] * (FLOPS[19] + FORCE_FLOPS[19] + ADJOINT_FLOPS)}
    q = 9 if kind in ("plane", "cavity") else 19
    flops = FLOPS[q] + (FORCE_FLOPS[q] if kind in ("channel", "plane", "restart") else 0)
    # a fifth of a sphere-filled channel is solid
    fluid = cells * (0.8 if kind in ("channel", "restart") else 1.0)
    if kind == "restart":
        return {"bytes": cells * 32 + fluid * 8 * q * 4, "flops": fluid * case["steps"] * flops}
    return {"bytes": fluid * 2 * q * BYTES[case["storage"]] + cells * 16,
            "flops": fluid * case["steps"] * flops}


# ---------------------------------------------------------------------------
# The same in 64 bits: two-lattice pull, one gather per population
# ---------------------------------------------------------------------------
def _velocities(q):
    """Velocities in the order the package documents for its populations, weights,
    opposites."""
    if q == 9:
        c = [(0, 0), (-1, 1), (-1, 0), (-1, -1), (0, -1), (1, -1), (1, 0), (1, 1), (0, 1)]
        c = [(x, y, 0) for x, y in c]
        w = {0: 16, 1: 4, 2: 1}
    else:
        h = [(-1, 0, 0), (0, -1, 0), (0, 0, -1), (-1, -1, 0), (-1, 1, 0), (-1, 0, -1), (-1, 0, 1),
             (0, -1, -1), (0, -1, 1)]
        c = [(0, 0, 0)] + h + [(-x, -y, -z) for x, y, z in h]
        w = {0: 12, 1: 2, 2: 1}
    return (c, [w[sum(v * v for v in k)] / 36 for k in c],
            [c.index((-x, -y, -z)) for x, y, z in c])


def _dot(c, v):
    """c.v of a lattice velocity and three fields (0 where c vanishes)."""
    r = 0.0
    for a, s in zip(v, c):
        if s:
            r = r + s * a
    return r


def _equilibrium(q, u):
    c, w, _ = _velocities(q)
    uu = (u * u).sum(0)
    f = torch.empty((q, u.shape[1]), dtype=torch.float64, device=u.device)
    for i in range(q):
        cu = _dot(c[i], u)
        f[i] = w[i] * (1 + 3 * cu + 4.5 * cu * cu - 1.5 * uu)
    return f


def _pull_index(q, mat, offset=0):
    """For population i of cell x, the place in the flattened (q, cells) array
    that it comes from: i at x - c_i, or its opposite at x across a wall."""
    c, _, opp = _velocities(q)
    m = torch.from_numpy(mat).to(DEVICE)
    n = m.numel()
    cell = torch.arange(n, device=DEVICE).reshape(m.shape)
    index = torch.empty((q, n), dtype=torch.int64, device=DEVICE)
    for i in range(q):
        shift = (c[i][2], c[i][1], c[i][0])
        wall = torch.roll(m, shift, (0, 1, 2)) >= 2
        index[i] = torch.where(wall, opp[i] * n + cell, i * n + torch.roll(cell, shift, (0, 1, 2))
                               ).reshape(-1)
    return index


def _moments64(q, f, g):
    c, _, _ = _velocities(q)
    rho = f.sum(0)
    u = torch.stack([sum(c[i][a] * f[i] for i in range(q) if c[i][a]) / rho + 0.5 * g[a]
                     if any(k[a] for k in c) else torch.zeros_like(rho) for a in range(3)])
    return rho, u


def _advance(q, f, index, omega, g, uw, moving, steps):
    c, w, opp = _velocities(q)
    forced, post = any(g), torch.empty_like(f)
    for _ in range(steps):
        rho, u = _moments64(q, f, g)
        uu = (u * u).sum(0)
        ug = sum(u[a] * g[a] for a in range(3))
        for i in range(q):
            cu = _dot(c[i], u)
            post[i] = f[i] - omega * (f[i] - w[i] * rho * (1 + 3 * cu + 4.5 * cu * cu - 1.5 * uu))
            if forced:
                cg = _dot(c[i], g)
                post[i] += (1 - 0.5 * omega) * w[i] * rho * (3 * (cg - ug) + 9 * cu * cg)
        for i in range(q):
            f[i] = post.reshape(-1)[index[i]]
            if moving is not None and _dot(c[i], uw):
                f[i] += moving[i] * (6 * w[i] * _dot(c[i], uw)) * rho
    return f


def _advance_porous(f, index, omega, g, d):
    """One step of the porous collision, differentiable in f and d."""
    c, w, _ = _velocities(19)
    cc = torch.tensor(c, dtype=torch.float64, device=DEVICE)
    ww = torch.tensor(w, dtype=torch.float64, device=DEVICE)[:, None]
    gg = torch.tensor(g, dtype=torch.float64, device=DEVICE)[:, None]
    rho = f.sum(0)
    v = d * (cc.T.contiguous() @ f / rho + 0.5 * gg)
    cv, cg = cc @ v, cc @ gg
    feq = ww * rho * (1 + 3 * cv + 4.5 * cv * cv - 1.5 * (v * v).sum(0))
    guo = (1 - 0.5 * omega) * ww * rho * (3 * (cg - (v * gg).sum(0)) + 9 * cv * cg)
    return (f - omega * (f - feq) + guo).reshape(-1)[index]


def _exact_adjoint(case, seed):
    mat, por, g = _porous(case, seed)
    omega, index = 1 / TAU["adjoint"], _pull_index(19, mat)
    fluid = torch.from_numpy(mat == 1).to(DEVICE).reshape(-1)
    d = torch.from_numpy(por).to(DEVICE).double().reshape(-1)
    f = _equilibrium(19, torch.zeros((3, mat.size), dtype=torch.float64, device=DEVICE))
    states = []
    for _ in range(case["steps"]):
        states.append(f)
        f = _advance_porous(f, index, omega, g, d)
    plane = fluid & (torch.arange(mat.size, device=DEVICE) % case["nx"] == case["nx"] - 1)
    f.requires_grad_()
    d.requires_grad_()
    objective = _moments64(19, f, g)[1][0][plane].mean()
    (lam,) = torch.autograd.grad(objective, f)
    grad = torch.zeros_like(d)
    while states:
        f = states.pop().requires_grad_()
        lam, part = torch.autograd.grad(_advance_porous(f, index, omega, g, d), (f, d),
                                        lam * fluid)
        grad += part
    return {"objective": objective.detach(), "grad": (grad * fluid).reshape(mat.shape)}


def _exact_ensemble(case, seed):
    shapes, tau = _ensemble(case, seed)
    rho, u = [], []
    for k, (shape, t) in enumerate(zip(shapes, tau)):
        mat = np.ones(tuple(reversed(shape)), np.uint8)
        f = _equilibrium(19, _flow(shape, seed + k).reshape(3, -1))
        f = _advance(19, f, _pull_index(19, mat), 1 / t, (0, 0, 0), (0, 0, 0), None,
                     case["steps"])
        r, v = _moments64(19, f, (0, 0, 0))
        rho.append(r)
        u.append(v)
    return {"rho": torch.cat(rho), "u": torch.cat(u, dim=1)}


def exact(case, seed):
    kind = case["kind"]
    if kind == "adjoint":
        return _exact_adjoint(case, seed)
    if kind == "ensemble":
        # every operation of a step is a launch of its own here: beyond a few
        # thousand lattice steps this takes too long
        return _exact_ensemble(case, seed) if case["count"] * case["steps"] <= 2000 else None
    problem = _problem(case, seed)
    q, mat, _, u, g, uw = problem
    n = mat.size
    if kind == "restart":
        f = _saved(problem, seed).reshape(q, -1)
    else:
        zero = torch.zeros((3, n), dtype=torch.float64, device=DEVICE)
        f = _equilibrium(q, zero if u is None else u.reshape(3, -1))
    index, moving = _pull_index(q, mat), None
    if any(uw):
        c, _, _ = _velocities(q)
        m = torch.from_numpy(mat).to(DEVICE)
        moving = [(torch.roll(m, (k[2], k[1], k[0]), (0, 1, 2)) == 3).reshape(-1) for k in c]
    fluid = torch.from_numpy(mat == 1).to(DEVICE)
    f = _advance(q, f, index, 1 / TAU[kind], g, uw, moving, case["steps"])
    rho, v = _moments64(q, f, g)
    keep = fluid.reshape(-1)
    rho = torch.where(keep, rho, 0.0)
    v = torch.where(keep, v, 0.0)
    if q == 9:
        v[2] = 0.0
    fields = {"rho": rho.reshape(mat.shape), "u": v.reshape(3, *mat.shape)}
    if kind != "restart":
        return fields
    f = torch.where(keep, f, 0.0)
    c, _, _ = _velocities(q)
    speed = (v * v).sum(0)
    count = int(keep.sum())
    return {"f": f.reshape(q, *mat.shape), "mass": float(rho.sum()),
            "momentum": np.array([float(sum(k[a] * f[i] for i, k in enumerate(c) if k[a]).sum())
                                  for a in range(3)]),
            "stats": np.array([float(rho.sum()) / count, 0.5 * float(speed.sum()) / count,
                               float(speed.max().sqrt())]),
            "rho": fields["rho"].cpu().numpy(), "u": fields["u"].cpu().numpy()}
