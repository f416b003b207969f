"""Workloads of the moving-mesh hydrodynamics path, through its public entry
points, from the smallest runs to the largest.

A case names an operation ("op"), an initial condition ("problem", one of
paper_1410_3219_amd.inputs) with k cells per side, and the options of the
scheme.  The operations:

  stage   one stage (rich_stage, or rich_stage_accel with "accel")
  pair    the two stages of a step on a static mesh, the Courant step taken on
          the device (rich_stage_courant, rich_stage_dt_of): what a served
          session with a static mesh asks for
  step    a whole time-centred step of a moving mesh on the device: stage 1,
          the mesh of the half-step points, stage 2, the mesh of the new ones
  retess  one rebuild of the mesh after the points have moved (rich_retess)
  driver  the Courant step read by the host, then rich_step with meshes built
          on the device: a program that advances one run step by step
  batch   both stages of many runs of uneven sizes, launched eagerly
          (rich_stage_batch): what the serving loop does on each tick
  plan    the same through prepared plans with each run's Courant step taken
          on the device (rich_stage_batch_prepare_courant once, then launches)
  sweep   one step of the cell-rounding parameter sweep (sweep.Sweep.step):
          many 30 x 30 runs on moving meshes
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_1410_3219_amd import inputs as I
from paper_1410_3219_amd import rich as R
from paper_1410_3219_amd import sweep as S
from paper_1410_3219_amd import tess as T


def listed():
    return [
        # one small vortex run, as the tests and the parameter sweep use it:
        # nothing but latency and launches
        _case("stage_gresho30", "stage", "gresho", 30),
        # a small shock tube between walls, exact solver, static mesh
        _case("pair_sod64_exact", "pair", "sod", 64, riemann=1, motion=0),
        # the same shock tube on a moving mesh, all of the step on the device
        _case("step_sod64", "step", "sod", 64),
        # a program that advances one odd-sized run step by step
        _case("driver_wave101", "driver", "wave", 101),
        # 16 runs of 900 cells advanced together, meshes rebuilt on the device
        _case("sweep_gresho30_x16", "sweep", "gresho", 30, runs=16),
        # a point explosion of a served session's size (static, ragged size)
        _case("pair_sedov181", "pair", "sedov", 181, motion=0),
        # many small independent shock tubes, plans prepared once
        _case("plan_sod_128_small", "plan", "sod", 0, runs=128, n_min=256, n_max=4096),
        # uneven shock tubes launched as the serving loop does
        _case("batch_sod_48", "batch", "sod", 0, runs=48, n_min=1024, n_max=65536),
        # a mesh between walls rebuilt after a move
        _case("retess_sod511", "retess", "sod", 511),
        # the one-stage integrator with an external acceleration field
        _case("stage_kh512_extrapolated", "stage", "kh", 512, integrator=1, accel=1),
        # the advected wave at a quarter of the benchmark's size, static mesh
        _case("pair_wave1024", "pair", "wave", 1024, motion=0),
        # the benchmark's workload: the 2048 x 2048 wave, a whole step
        _case("step_wave2048", "step", "wave", 2048),
    ]


def draw(rng):
    op = rng.choice(["stage", "stage", "pair", "pair", "step", "step", "step", "retess", "retess",
                     "driver", "batch", "plan", "sweep"])
    if op == "sweep":
        return _case("", op, "gresho", 30, runs=rng.randint(2, 30), salt=rng.randrange(1 << 20))
    if op in ("batch", "plan"):
        n_min = int(round(math.exp(rng.uniform(math.log(64), math.log(4096)))))
        runs = int(round(math.exp(rng.uniform(math.log(2), math.log(160)))))
        n_max = int(n_min * math.exp(rng.uniform(0.0, math.log(32))))
        runs = max(2, min(runs, int(1.0e6 / math.sqrt(n_min * n_max))))   # about a million cells
        return _case("", op, "sod", 0, runs=runs, n_min=n_min, n_max=n_max,
                     riemann=int(rng.random() < 0.2), salt=rng.randrange(1 << 20))
    hi = {"driver": 300, "step": 1100, "retess": 1100, "stage": 1100, "pair": 1100}[op]
    k = int(round(math.exp(rng.uniform(math.log(10), math.log(hi)))))
    # (a driven run goes on from pass to pass: smooth flows, for any number of steps)
    problem = rng.choice(["wave", "gresho"] if op == "driver" else ["sod", "wave", "gresho", "kh"])
    if op in ("stage", "pair") and k <= 400 and rng.random() < 0.2:
        problem = "sedov"
    opt = {"riemann": int(rng.random() < 0.25), "salt": rng.randrange(1 << 20)}
    if op == "stage":
        opt["integrator"] = int(rng.random() < 0.25)
        opt["accel"] = int(rng.random() < 0.25)
        opt["limiter"] = rng.choice([0, 0, 0, 1, 2, 4])
    if op in ("stage", "pair"):
        opt["motion"] = 1 if op == "stage" and rng.random() < 0.7 else 0
    return _case("", op, problem, k, **opt)


def _case(name, op, problem, k, **opt):
    c = {"name": name} if name else {}
    c.update(op=op, problem=problem, k=k, riemann=0, motion=1, integrator=0, limiter=0, accel=0,
             runs=0, n_min=0, n_max=0, salt=0)
    c.update(opt)
    return c


# ---------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------
MAKE = {"sod": I.sod, "wave": I.advected_wave, "gresho": I.gresho, "kh": I.kelvin_helmholtz,
        "sedov": I.sedov}


def _problem(name, k, seed, angle=None, gamma=None):
    kw = {"k": k, "seed": 1 + 7919 * seed}
    if angle is not None:
        kw["angle"] = angle
    if gamma is not None:
        kw["gamma"] = gamma
    return MAKE[name](**kw)


def _host(P):
    """Mesh, conserved totals and points of a problem, on the host."""
    m = T.rich_tess_build(P.px, P.py, P.box, P.bc)
    Q = I.sedov_state(P, m.area) if P.name == "sedov" else P.state(m.area)
    return m, Q, np.stack([m.px, m.py])


def _params(case, gamma, **kw):
    return R.Params(gamma=gamma, riemann=case["riemann"], motion=case["motion"],
                    limiter=case["limiter"], integrator=case["integrator"], **kw)


def _half_step(m, Q, gamma):
    """Half a Courant step of the state at rest in the box's frame."""
    rho, vx, vy, p = _prims(Q, m.area, gamma)
    c = np.sqrt(gamma * p / rho) + np.hypot(vx, vy)
    return 0.15 * float(np.min(np.sqrt(m.area / math.pi) / c))


def _moved(m, X, seed):
    """The points after a half step: a common drift and a small change of each
    (in lattice spacings, of the size that the benchmark's wave shows)."""
    h = math.sqrt((m.box[2] - m.box[0]) * (m.box[3] - m.box[1]) / m.n_cells)
    g = np.random.default_rng(seed + 77)
    d = g.uniform(-0.02, 0.02, X.shape)
    if m.bc == T.BC_PERIODIC:
        d += np.array([[0.075], [0.0375]])
    Y = X + h * d
    for a in (0, 1):
        lo, hi = m.box[a], m.box[2 + a]
        if m.bc == T.BC_PERIODIC:
            Y[a] = lo + np.mod(Y[a] - lo, hi - lo)
        else:
            Y[a] = np.clip(Y[a], lo + 1e-3 * h, hi - 1e-3 * h)
    return Y


def _accel(n, seed):
    return np.random.default_rng(seed + 99).uniform(-0.1, 0.1, (2, n))


def _runs(case, seed):
    """Problems and rounding strengths of a batch (the case says the sizes)."""
    return [(_problem("sod", r["side"], seed * 1000 + r["seed"], angle=r["angle"],
                      gamma=r["gamma"]), r["chi"]) for r in _sizes(case)]


def _sizes(case):
    return I.batch_runs(case["runs"], seed=17 + case["salt"], n_min=case["n_min"],
                        n_max=case["n_max"])


class _State:
    pass


def _flat_states(ns):
    """States of many runs in one buffer (so that they can be returned whole)."""
    flat = torch.zeros(6 * sum(ns), dtype=torch.float64, device="cuda")
    out, o = [], 0
    for n in ns:
        out.append(R.DeviceState(flat[o:o + 4 * n].view(4, n), flat[o + 4 * n:o + 6 * n].view(2, n)))
        o += 6 * n
    return flat, out


def _mesh_out(b):
    """The written parts of a rebuilt mesh's buffers, by type."""
    e = b.t["edges"]
    e.zero_()
    return {"cells": b.t["cells"].view(torch.float64).view(-1, 6)[:, :5],
            "edges": e.view(torch.float64).view(-1, 4)[:, :3],
            "ij": e.view(torch.int32).view(-1, 8)[:, 6:],
            "off": b.t["off"], "idx": b.t["idx"], "eoff": b.t["eoff"]}


def prepare(case, seed):
    seed = seed % (1 << 20) + case["salt"]
    op, s = case["op"], _State()
    s.op = op
    if op == "sweep":
        g = S.chi_eta_grid(4, 8)
        s.sweep = S.Sweep(g[:case["runs"]], k=case["k"], seed=4 + seed, device_tess=True)
        s.out = {"Q": [x.Q for x in s.sweep.states], "X": [x.X for x in s.sweep.states]}
        return s
    if op in ("batch", "plan"):
        hosts = [(_host(P), P.gamma, chi) for P, chi in _runs(case, seed)]
        s.meshes = [R.DeviceMesh.from_host(h[0]) for h, _, _ in hosts]
        s.cur = [R.DeviceState.from_host(h[1], h[2]) for h, _, _ in hosts]
        ns = [m.n_cells for m in s.meshes]
        s.half_flat, s.half = _flat_states(ns)
        s.next_flat, s.next = _flat_states(ns)
        s.params = [_params(case, g, chi=chi) for _, g, chi in hosts]
        s.h = [_half_step(h[0], h[1], g) for h, g, _ in hosts]
        s.h2 = [2.0 * h for h in s.h]
        s.ws, s.ws2 = R.batch_workspace(ns), R.batch_workspace(ns)
        if op == "plan":
            n = len(ns)
            s.plan1 = R.rich_stage_batch_prepare_courant(s.meshes, s.cur, s.cur, s.half, [0.5] * n,
                                                         s.params, s.ws)
            s.plan2 = R.rich_stage_batch_prepare_courant(s.meshes, s.half, s.cur, s.next, [1.0] * n,
                                                         s.params, s.ws2, dt_ws=s.ws)
        s.out = {"half": s.half_flat, "next": s.next_flat}
        return s
    P = _problem(case["problem"], case["k"], seed)
    m, Q, X = _host(P)
    n = m.n_cells
    s.params = _params(case, P.gamma)
    if op == "driver":
        s.ctx = R.RichCtx(device_tess=True)
        s.ctx.set_mesh(m)
        s.cur = R.DeviceState.from_host(Q, X)
        s.ws = R.workspace(n)
        return s
    s.mesh = R.DeviceMesh.from_host(m)
    if op == "retess":
        s.X = torch.from_numpy(_moved(m, X, seed)).cuda()
        s.bufs = R.DeviceMeshBufs(n, m.box, m.bc)
        s.rws = R.retess_workspace(n)
        s.out = _mesh_out(s.bufs)
        return s
    s.cur = R.DeviceState.from_host(Q, X)
    s.half, s.next = R.DeviceState.empty_like(s.cur), R.DeviceState.empty_like(s.cur)
    s.ws = R.workspace(n)
    if op == "stage":
        s.h = _half_step(m, Q, P.gamma)
        s.accel = torch.from_numpy(_accel(n, seed)).cuda() if case["accel"] else None
        s.out = {"Q": s.half.Q, "X": s.half.X}
    elif op == "pair":
        s.out = {"Qh": s.half.Q, "Xh": s.half.X, "Q": s.next.Q, "X": s.next.X}
    else:
        s.b1, s.b2 = (R.DeviceMeshBufs(n, m.box, m.bc) for _ in range(2))
        s.m1 = s.b1.mesh()
        s.rws = R.retess_workspace(n)
        s.out = {"Q": s.next.Q, "X": s.next.X, "mesh1": _mesh_out(s.b1), "mesh2": _mesh_out(s.b2)}
    return s


def run(s):
    op = s.op
    if op == "stage":
        if s.accel is None:
            R.rich_stage(s.mesh, s.cur, s.cur, s.half, s.h, s.params, s.ws)
        else:
            R.rich_stage_accel(s.mesh, s.cur, s.cur, s.half, s.h, s.params, s.accel, s.ws)
    elif op == "pair":
        R.rich_stage_courant(s.mesh, s.cur, s.cur, s.half, 0.5, s.params, s.ws)
        R.rich_stage_dt_of(s.mesh, s.half, s.cur, s.next, 1.0, s.ws, s.params, s.ws)
    elif op == "step":
        R.rich_stage_courant(s.mesh, s.cur, s.cur, s.half, 0.5, s.params, s.ws)
        R.rich_retess(s.mesh, s.half.X, s.b1, s.rws)
        R.rich_stage_dt_of(s.m1, s.half, s.cur, s.next, 1.0, s.ws, s.params, s.ws)
        R.rich_retess(s.m1, s.next.X, s.b2, s.rws)
    elif op == "retess":
        R.rich_retess(s.mesh, s.X, s.bufs, s.rws)
    elif op == "driver":
        dt = R.rich_cfl_dt(s.ctx.mesh(), s.cur, s.params, s.ws)
        s.ctx.step(s.cur, dt, s.params)
        return {"dt": dt, "Q": s.cur.Q, "X": s.cur.X}
    elif op == "batch":
        R.rich_stage_batch(s.meshes, s.cur, s.cur, s.half, s.h, s.params, s.ws)
        R.rich_stage_batch(s.meshes, s.half, s.cur, s.next, s.h2, s.params, s.ws2)
    elif op == "plan":
        R.rich_stage_batch_launch(s.plan1, s.ws)
        R.rich_stage_batch_launch(s.plan2, s.ws2)
    else:
        s.sweep.step()
    return s.out


def _cells(case):
    if case["op"] in ("batch", "plan"):
        return sum(r["side"] ** 2 for r in _sizes(case))
    return case["k"] ** 2 * max(1, case["runs"])


def work(case):
    """Per cell (3 edges, 6 CSR entries): a stage reads the cell (40 B), its
    totals (32 B), edges (96 B) and CSR (28 B) and writes the new totals and
    point (48 B); the second stage also reads the base state (48 B).  A
    rebuild reads the points (16 B) and the previous CSR and edges (124 B) and
    writes cells, edges and CSR (168 B)."""
    n, op = _cells(case), case["op"]
    one, two, mesh = 244, 292, 308
    fl, fm = 1000 + (3000 if case["riemann"] else 0), 300
    b, f = {"stage": (one + 16 * case["accel"], fl), "retess": (mesh, fm),
            "pair": (one + two, 2 * fl), "batch": (one + two, 2 * fl), "plan": (one + two, 2 * fl),
            }.get(op, (one + two + 2 * mesh, 2 * (fl + fm)))
    return {"bytes": b * n, "flops": f * n}


# ---------------------------------------------------------------------------
# the same in plain numpy
# ---------------------------------------------------------------------------
def _prims(Q, area, gamma):
    rho = Q[0] / area
    vx, vy = Q[1] / Q[0], Q[2] / Q[0]
    return rho, vx, vy, (gamma - 1.0) * (Q[3] / area - 0.5 * rho * (vx * vx + vy * vy))


def _shift(code, box):
    k = np.where(code <= 4, code - 1, code)
    img = (code >= 1) & (code <= 8)
    return (np.where(img, k // 3 - 1, 0) * (box[2] - box[0]),
            np.where(img, k % 3 - 1, 0) * (box[3] - box[1]))


def _mirror(code, x, y, box):
    x = np.where(code == 9, 2 * box[0] - x, np.where(code == 10, 2 * box[2] - x, x))
    return x, np.where(code == 11, 2 * box[1] - y, np.where(code == 12, 2 * box[3] - y, y))


def _velocity(m, Q, p):
    """Point velocities with the cell-rounding correction, and the Courant minimum."""
    rho, vx, vy, pr = _prims(Q, m.area, p.gamma)
    c, rad = np.sqrt(p.gamma * pr / rho), np.sqrt(m.area / math.pi)
    wx, wy = np.zeros_like(vx), np.zeros_like(vy)
    if p.motion:
        dx, dy = m.sx - m.px, m.sy - m.py
        d = np.hypot(dx, dy)
        on = d > p.eta * rad
        f = np.where(on, p.chi * c / np.where(on, d, 1.0), 0.0)
        wx, wy = vx + f * dx, vy + f * dy
    return c, rad, wx, wy, float(np.min(rad / (c + np.hypot(vx - wx, vy - wy))))


def _stage(m, Qs, Qb, Xb, h, p, accel=None):
    n, box = m.n_cells, m.box
    phi = np.stack(_prims(Qs, m.area, p.gamma))
    c, rad, wx, wy, _ = _velocity(m, Qs, p)
    # neighbours across the CSR entries
    row = np.repeat(np.arange(n), np.diff(m.off))
    e, side = m.idx >> 1, (m.idx & 1) == 1
    nb, code = m.nb_cell(), m.nb_code()
    sx, sy = _shift(code, box)
    wall = ~side & (code[e] >= 9)
    j = np.where(side, m.e_i[e], np.where(wall, row, nb[e]))
    ex, ey = np.where(side, -sx[e], sx[e]), np.where(side, -sy[e], sy[e])
    mx, my = _mirror(code[e], m.px[row], m.py[row], box)
    rjx, rjy = np.where(wall, mx, m.px[j] + ex), np.where(wall, my, m.py[j] + ey)
    fx, fy = m.e_fx[e] + np.where(side, ex, 0.0), m.e_fy[e] + np.where(side, ey, 0.0)
    pj = phi[:, j].copy()
    pj[1] = np.where(wall & (code[e] <= 10), -pj[1], pj[1])
    pj[2] = np.where(wall & (code[e] >= 11), -pj[2], pj[2])
    # gradient
    rx, ry = m.px[row] - rjx, m.py[row] - rjy
    lr = m.e_len[e] / np.hypot(rx, ry)
    cx, cy = fx - 0.5 * (m.px[row] + rjx), fy - 0.5 * (m.py[row] + rjy)
    G = np.empty((4, 2, n))
    for q in range(4):
        d, a = pj[q] - phi[q][row], 0.5 * (pj[q] + phi[q][row])
        G[q, 0] = np.bincount(row, lr * (d * cx - a * rx), n) / m.area
        G[q, 1] = np.bincount(row, lr * (d * cy - a * ry), n) / m.area
    # limiter
    at = m.off[:-1]
    jump = np.minimum(phi[3][row], pj[3]) < p.delta_p * np.maximum(phi[3][row], pj[3])
    shock = np.logical_or.reduceat(jump, at) | (-(G[1, 0] + G[2, 1]) * rad > p.delta_v * c)
    local = {0: shock, 1: np.zeros(n, bool), 2: np.ones(n, bool)}.get(p.limiter)
    L = G.copy()
    for q in range(4):
        hi = np.maximum(phi[q], np.maximum.reduceat(pj[q], at))
        lo = np.minimum(phi[q], np.minimum.reduceat(pj[q], at))
        d = G[q, 0][row] * (fx - m.sx[row]) + G[q, 1][row] * (fy - m.sy[row])
        dd, f = np.where(d == 0, 1.0, d), phi[q][row]
        wide = np.where(d > 0, (hi[row] - f) / dd, np.where(d < 0, (lo[row] - f) / dd, 1.0))
        near = np.where(d == 0, 1.0, np.maximum(p.theta * (pj[q] - f) / dd, 0.0))
        if p.limiter == 4:
            L[q] = 0.0
        elif local is not None:
            L[q] *= np.minimum(1.0, np.minimum.reduceat(np.where(local[row], near, wide), at))
    if p.integrator == 1:
        rho, vx, vy, pr = phi
        ux, uy, div = vx - wx, vy - wy, L[1, 0] + L[2, 1]
        t = np.stack([-(ux * L[0, 0] + uy * L[0, 1]) - rho * div,
                      -(ux * L[1, 0] + uy * L[1, 1]) - L[3, 0] / rho,
                      -(ux * L[2, 0] + uy * L[2, 1]) - L[3, 1] / rho,
                      -(ux * L[3, 0] + uy * L[3, 1]) - p.gamma * pr * div])
        phi = phi + 0.5 * h * t
    # fluxes
    i, wl = m.e_i, code >= 9
    k = np.where(wl, i, nb)
    left = phi[:, i] + L[:, 0, i] * (m.e_fx - m.sx[i]) + L[:, 1, i] * (m.e_fy - m.sy[i])
    right = (phi[:, k] + L[:, 0, k] * (m.e_fx - sx - m.sx[k]) +
             L[:, 1, k] * (m.e_fy - sy - m.sy[k]))
    wix, wiy, wkx, wky = wx[i], wy[i], wx[k], wy[k]
    mx, my = _mirror(code, m.px[i], m.py[i], box)
    kx, ky = np.where(wl, mx, m.px[k] + sx), np.where(wl, my, m.py[k] + sy)
    vert, flat = wl & (code <= 10), wl & (code >= 11)
    wkx, wky = np.where(vert, -wkx, wkx), np.where(flat, -wky, wky)
    right = np.where(wl, left, right)
    right[1], right[2] = np.where(vert, -right[1], right[1]), np.where(flat, -right[2], right[2])
    dx, dy = kx - m.px[i], ky - m.py[i]
    d = np.hypot(dx, dy)
    nx, ny = dx / d, dy / d
    cx, cy = m.e_fx - 0.5 * (m.px[i] + kx), m.e_fy - 0.5 * (m.py[i] + ky)
    a = np.where(wl, 0.0, ((wix - wkx) * cx + (wiy - wky) * cy) / d)
    vx, vy = 0.5 * (wix + wkx) + a * nx, 0.5 * (wiy + wky) + a * ny
    vx, vy = np.where(flat, wix, np.where(vert, 0.0, vx)), np.where(vert, wiy, np.where(flat, 0.0, vy))
    W = []
    for s in (left, right):
        ux, uy = s[1] - vx, s[2] - vy
        W.append((s[0], ux * nx + uy * ny, uy * nx - ux * ny, s[3]))
    F = (_exact_flux if p.riemann else _hllc)(p.gamma, *W)
    px, py = F[1] * nx - F[2] * ny, F[1] * ny + F[2] * nx
    F = np.stack([F[0], px + F[0] * vx, py + F[0] * vy,
                  F[3] + px * vx + py * vy + 0.5 * (vx * vx + vy * vy) * F[0]]) * m.e_len
    sign = np.where(side, -1.0, 1.0)
    Q = np.stack([Qb[q] - h * np.bincount(row, sign * F[q][e], n) for q in range(4)])
    if accel is not None:
        Q[1] += h * Qs[0] * accel[0]
        Q[2] += h * Qs[0] * accel[1]
        Q[3] += h * (Qs[1] * accel[0] + Qs[2] * accel[1])
    X = Xb + h * np.stack([wx, wy])
    if m.bc == T.BC_PERIODIC:
        for q in (0, 1):
            lo, hi = box[q], box[q + 2]
            X[q] = np.where(X[q] < lo, X[q] + (hi - lo), X[q])
            X[q] = np.where(X[q] >= hi, X[q] - (hi - lo), X[q])
    return Q, X


def _flux(g, W):
    rho, u, v, p = W
    return np.stack([rho * u, rho * u * u + p, rho * u * v,
                     u * (p / (g - 1) + 0.5 * rho * (u * u + v * v) + p)])


def _hllc(g, l, r):
    cl, cr = np.sqrt(g * l[3] / l[0]), np.sqrt(g * r[3] / r[0])
    sl, sr = np.minimum(l[1] - cl, r[1] - cr), np.maximum(l[1] + cl, r[1] + cr)
    ss = ((r[3] - l[3] + l[0] * l[1] * (sl - l[1]) - r[0] * r[1] * (sr - r[1])) /
          (l[0] * (sl - l[1]) - r[0] * (sr - r[1])))
    star = []
    for (rho, u, v, p), s in ((l, sl), (r, sr)):
        E = p / (g - 1) + 0.5 * rho * (u * u + v * v)
        rs = rho * (s - u) / (s - ss)
        ps = p + rho * (s - u) * (ss - u)
        Es = rs * (E / rho + (ss - u) * (ss + p / (rho * (s - u))))
        star.append(np.stack([rs * ss, rs * ss * ss + ps, rs * ss * v, (Es + ps) * ss]))
    return np.where(sl >= 0, _flux(g, l),
                    np.where(ss >= 0, star[0], np.where(sr > 0, star[1], _flux(g, r))))


def _exact_flux(g, l, r):
    """Godunov flux of the exact Riemann problem (Newton iterations on the star pressure)."""
    def side(ps, W, c):
        A, B = 2 / ((g + 1) * W[0]), (g - 1) / (g + 1) * W[3]
        q = np.sqrt(A / (ps + B))
        x = ps / W[3]
        hit = ps > W[3]
        return (np.where(hit, (ps - W[3]) * q, 2 * c / (g - 1) * (x ** ((g - 1) / (2 * g)) - 1)),
                np.where(hit, q * (1 - 0.5 * (ps - W[3]) / (B + ps)),
                         x ** (-(g + 1) / (2 * g)) / (W[0] * c)))
    cl, cr = np.sqrt(g * l[3] / l[0]), np.sqrt(g * r[3] / r[0])
    ps = np.maximum(0.5 * (l[3] + r[3]) - 0.125 * (r[1] - l[1]) * (l[0] + r[0]) * (cl + cr), 1e-14)
    for _ in range(60):
        (fl, dl), (fr, dr) = side(ps, l, cl), side(ps, r, cr)
        was, ps = ps, np.maximum(ps - (fl + fr + r[1] - l[1]) / (dl + dr), 1e-14)
        if np.max(np.abs(ps - was) / ps) < 1e-15:
            break
    fl, fr = side(ps, l, cl)[0], side(ps, r, cr)[0]
    us = 0.5 * (l[1] + r[1]) + 0.5 * (fr - fl)
    out = []
    for W, c, sg in ((l, cl, 1.0), (r, cr, -1.0)):   # the right side mirrored
        rho, u, p = W[0], sg * W[1], W[3]
        U, x, g6 = sg * us, ps / W[3], (g - 1) / (g + 1)
        with np.errstate(invalid="ignore"):
            shock = u - c * np.sqrt((g + 1) / (2 * g) * x + (g - 1) / (2 * g))
            cs = c * x ** ((g - 1) / (2 * g))
            cc = 2 / (g + 1) * (c + (g - 1) / 2 * u)
            fan = (rho * np.maximum(cc / c, 0) ** (2 / (g - 1)), cc,
                   p * np.maximum(cc / c, 0) ** (2 * g / (g - 1)))
        hit = ps > p
        keep = np.where(hit, shock >= 0, u - c >= 0)
        star = np.where(hit, True, U - cs < 0)
        sr = np.where(hit, rho * (x + g6) / (g6 * x + 1), rho * x ** (1 / g))
        d = np.where(keep, rho, np.where(star, sr, fan[0]))
        v = np.where(keep, u, np.where(star, U, fan[1]))
        q = np.where(keep, p, np.where(star, ps, fan[2]))
        out.append(_flux(g, (d, sg * v, W[2], q)))
    return np.where(us >= 0, out[0], out[1])


class _Mesh:
    """The mesh fields that _stage reads."""
    nb_cell, nb_code = T.HostMesh.nb_cell, T.HostMesh.nb_code


def _voronoi(X, box, bc, K=30):
    """Voronoi mesh of points of about even spacing: each point's bisectors
    with its K nearest images (and its mirrors) cut down by one another."""
    n = X.shape[1]
    L = np.array([box[2] - box[0], box[3] - box[1]])
    lo = np.array([box[0], box[1]])
    # points in square bins of about one point each, searched three bins wide
    k = np.maximum(1, np.floor(L / math.sqrt(L[0] * L[1] / n)).astype(int))
    b = np.minimum(((X.T - lo) / L * k).astype(int), k - 1)
    flat = b[:, 0] * k[1] + b[:, 1]
    order = np.argsort(flat, kind="stable")
    start = np.searchsorted(flat[order], np.arange(k[0] * k[1] + 1))
    most = int(np.max(np.diff(start)))
    ids, codes, ds = [], [], []
    for ox in range(-3, 4):
        for oy in range(-3, 4):
            u = b + [ox, oy]
            turn = np.floor_divide(u, k)
            in_box = (turn == 0).all(1) if bc == T.BC_WALLS else np.ones(n, bool)
            v = np.mod(u, k)
            cell = v[:, 0] * k[1] + v[:, 1]
            s = (turn[:, 0] + 1) * 3 + turn[:, 1] + 1
            code = np.where(s == 4, 0, np.where(s < 4, s + 1, s))
            for q in range(most):
                at = start[cell] + q
                ok = in_box & (at < start[cell + 1])
                j = order[np.minimum(at, n - 1)]
                d = X[:, j].T + turn * L - X.T
                ok &= ~((j == np.arange(n)) & (code == 0))
                ids.append(j)
                codes.append(code)
                ds.append(np.where(ok[:, None], d, 1e9))
    ids, codes, ds = np.stack(ids, 1), np.stack(codes, 1), np.stack(ds, 1)
    near = np.argsort((ds ** 2).sum(2), 1)[:, :K]
    take = lambda v: np.take_along_axis(v, near, 1)   # noqa: E731
    ids, codes = take(ids), take(codes)
    dx, dy = take(ds[:, :, 0]), take(ds[:, :, 1])
    if bc == T.BC_WALLS:
        z, own = np.zeros(n), np.arange(n)
        for cd, mx, my in ((9, 2 * (box[0] - X[0]), z), (10, 2 * (box[2] - X[0]), z),
                           (11, z, 2 * (box[1] - X[1])), (12, z, 2 * (box[3] - X[1]))):
            ids, codes = np.c_[ids, own], np.c_[codes, np.full(n, cd)]
            dx, dy = np.c_[dx, mx], np.c_[dy, my]
    hh = 0.5 * (dx * dx + dy * dy)
    K = dx.shape[1]
    t0, t1 = np.full((n, K), -np.inf), np.full((n, K), np.inf)
    with np.errstate(divide="ignore", invalid="ignore"):
        for v in range(K):
            a = -dy * dx[:, v:v + 1] + dx * dy[:, v:v + 1]
            t = (hh[:, v:v + 1] - 0.5 * (dx * dx[:, v:v + 1] + dy * dy[:, v:v + 1])) / a
            a[:, v] = 0.0
            t1 = np.where(a > 0, np.minimum(t1, t), t1)
            t0 = np.where(a < 0, np.maximum(t0, t), t0)
    live = t0 < t1
    r, c = np.nonzero(live)
    ang = np.mod(np.arctan2(dy[r, c], dx[r, c]), 2 * math.pi)
    o = np.lexsort((ang, r))
    r, c = r[o], c[o]
    dx, dy, t0, t1, ids, codes = (v[r, c] for v in (dx, dy, t0, t1, ids, codes))
    ux, uy, vx, vy = 0.5 * dx - t0 * dy, 0.5 * dy + t0 * dx, 0.5 * dx - t1 * dy, 0.5 * dy + t1 * dx
    cr = ux * vy - uy * vx
    A = np.bincount(r, cr, n)
    m = _Mesh()
    m.n_cells, m.box, m.bc = n, box, bc
    m.px, m.py, m.area = X[0], X[1], 0.5 * A
    m.sx = X[0] + np.bincount(r, (ux + vx) * cr, n) / (3 * A)
    m.sy = X[1] + np.bincount(r, (uy + vy) * cr, n) / (3 * A)
    own = (codes >= 9) | (r < ids) | ((r == ids) & (codes >= 5))
    m.e_i = r[own].astype(np.int32)
    m.e_j = (ids[own].astype(np.uint32) | (codes[own].astype(np.uint32) << 28)).view(np.int32)
    m.e_len = np.hypot(vx - ux, vy - uy)[own]
    m.e_fx, m.e_fy = (X[0][r] + 0.5 * (ux + vx))[own], (X[1][r] + 0.5 * (uy + vy))[own]
    # CSR: each entry's edge, found by its two cells and the image between them
    m.off = np.concatenate([[0], np.cumsum(np.bincount(r, minlength=n))]).astype(np.int32)
    back = np.where((codes >= 1) & (codes <= 8), 9 - codes, codes)
    key = np.where(own, (r * n + ids) * 16 + codes, (ids * n + r) * 16 + back)
    srt = np.argsort(key[own])
    m.idx = (2 * srt[np.searchsorted(key[own], key, sorter=srt)] + ~own).astype(np.int32)
    return m


def _mesh_exact(m):
    ce, _ = R.rich_retess_capacity(m.n_cells)
    e = np.zeros((ce, 3))
    e[:len(m.e_len)] = np.stack([m.e_fx, m.e_fy, m.e_len], 1)
    return {"cells": np.stack([m.px, m.py, m.area, m.sx, m.sy], 1), "edges": e,
            "ij": None, "off": None, "idx": None, "eoff": None}


def _step(m, Q, X, p, courant=0.3):
    dt = courant * _velocity(m, Q, p)[4]
    Qh, Xh = _stage(m, Q, Q, X, 0.5 * dt, p)
    mh = _voronoi(Xh, m.box, m.bc)
    return (dt, mh) + _stage(mh, Qh, Q, X, dt, p)


def exact(case, seed):
    with np.errstate(all="ignore"):
        return _exact(case, seed)


def _exact(case, seed):
    seed = seed % (1 << 20) + case["salt"]
    op, n = case["op"], _cells(case)
    most = 700000 // (1 + 2 * case["riemann"]) if op in ("stage", "pair", "batch", "plan") else 20000
    if n > most:
        return None   # over about 20 seconds
    if op == "sweep":
        P = I.gresho(k=case["k"], seed=4 + seed)
        m, Q, X = _host(P)
        out = [_step(m, Q, X, R.Params(gamma=P.gamma, chi=c, eta=e))[2:]
               for c, e in S.chi_eta_grid(4, 8)[:case["runs"]]]
        return {"Q": [q for q, _ in out], "X": [x for _, x in out]}
    if op in ("batch", "plan"):
        half, last = [], []
        for P, chi in _runs(case, seed):
            m, Q, X = _host(P)
            p = _params(case, P.gamma, chi=chi)
            h = 0.15 * _velocity(m, Q, p)[4] if op == "plan" else _half_step(m, Q, P.gamma)
            Qh, Xh = _stage(m, Q, Q, X, h, p)
            Qn, Xn = _stage(m, Qh, Q, X, 2 * h, p)
            half += [Qh.ravel(), Xh.ravel()]
            last += [Qn.ravel(), Xn.ravel()]
        return {"half": np.concatenate(half), "next": np.concatenate(last)}
    P = _problem(case["problem"], case["k"], seed)
    m, Q, X = _host(P)
    p = _params(case, P.gamma)
    if op == "stage":
        Q1, X1 = _stage(m, Q, Q, X, _half_step(m, Q, P.gamma), p,
                        _accel(m.n_cells, seed) if case["accel"] else None)
        return {"Q": Q1, "X": X1}
    if op == "pair":
        dt = 0.3 * _velocity(m, Q, p)[4]
        Qh, Xh = _stage(m, Q, Q, X, 0.5 * dt, p)
        Qn, Xn = _stage(m, Qh, Q, X, dt, p)
        return {"Qh": Qh, "Xh": Xh, "Q": Qn, "X": Xn}
    if op == "retess":
        return _mesh_exact(_voronoi(_moved(m, X, seed), m.box, m.bc))
    dt, mh, Qn, Xn = _step(m, Q, X, p)
    if op == "driver":
        return {"dt": dt, "Q": Qn, "X": Xn}
    return {"Q": Qn, "X": Xn, "mesh1": _mesh_exact(mh),
            "mesh2": _mesh_exact(_voronoi(Xn, m.box, m.bc))}
