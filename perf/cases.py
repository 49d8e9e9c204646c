"""Timed cases of the library: grid runs, ensembles, training and state output.

Every case is what a program written against the binding does with states that
are already on the GPU.  `listed()` gives the fixed cases, `draw(rng)` one more
of the same ranges, `prepare` the inputs and handles, `run` one pass, `work`
the bytes and operations a pass cannot do without, and `exact` the same result
from plain float64 torch, evaluated as the formulas are printed.
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2208_04488_amd import hrm, learned

P0, T0, TRACE = 101325.0, 298.0, 1e-8
LIQUID_A, LIQUID_B = (4.4, 4200.0, 6e8), (6.12, 4200.0, 3.43e8)  # gamma, c_p, p_inf
AIR, LIGHT = (1.4, 1007.0, 0.0), (1.67, 5193.0, 0.0)
OPEN, PERIODIC, INFLOW = hrm.BC_TRANSMISSIVE, hrm.BC_PERIODIC, hrm.BC_DIRICHLET
CFL = 0.4


def listed():
    return [
        # one shock tube on a line, run to its end time in chunks of steps: the smallest grid there is
        grid("tube_400", (400,), 2, steps=50),
        # the comparison scheme (first order, four equations) at the ten times finer line it needs
        grid("tube_four_eq_5000", (5000,), 2, steps=20, scheme="four_eq"),
        # a small two-dimensional run under the caller's own time loop (wavespeed, time step, three stages)
        grid("plane_127x65_stages", (127, 65), 2, call="stages", bounds="periodic"),
        # shock on a liquid column, three species: the ordinary two-dimensional run, both face precisions
        grid("column_1024x512", (1024, 512), 3, steps=5),
        grid("column_1024x512_fp32", (1024, 512), 3, steps=2, precision="fp32"),
        # a jet entering through a boundary with a set state, a grid width that no tile divides
        grid("jet_1000x500", (1000, 500), 2, steps=5, bounds="inflow"),
        # the largest grid of the benchmark: three dimensions, three species
        grid("multimode_256x256x256", (256, 256, 256), 3, steps=2, bounds="mixed"),
        # learned interpolation weights on a planar shock tube
        grid("learned_1024x512", (1024, 512), 2, steps=2, weights="mlp"),
        # thousands of independent shock tubes of different lengths
        ensemble("ensemble_4096", 4096, 200, 2000, 2, 10),
        # a few hundred short ones with float faces: fewer problems than the chip has room for
        ensemble("ensemble_300_fp32", 300, 40, 400, 2, 10, precision="fp32"),
        # a few optimiser steps on the interpolation weights
        dict(name="training_16384", kind="train", pairs=1 << 20, batch=16384, steps=5),
        # relaxing a state and writing out p, T, c and the wavespeeds
        dict(name="output_2048x1280", kind="output", n0=2048, n1=1280, n2=1, dim=2, species=2),
    ]


def grid(name, n, species, steps=1, precision="fp64", scheme="wcns", weights="is", bounds="open", call="advance"):
    c = dict(kind="grid", dim=len(n), n0=n[0], n1=n[1] if len(n) > 1 else 1, n2=n[2] if len(n) > 2 else 1,
             species=species, steps=steps, precision=precision, scheme=scheme, weights=weights, bounds=bounds, call=call)
    return dict(c, name=name) if name else c


def ensemble(name, problems, shortest, longest, species, steps, precision="fp64"):
    c = dict(kind="ensemble", problems=problems, shortest=shortest, longest=longest, species=species, steps=steps,
             precision=precision)
    return dict(c, name=name) if name else c


def draw(rng):
    def size(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    kind = rng.choice(["line", "plane", "plane", "cube", "cube", "ensemble", "ensemble", "train", "output"])
    sp, prec = rng.choice([2, 3]), rng.choice(["fp64", "fp64", "fp32"])
    if kind == "line":
        return grid(None, (size(100, 20000),), sp, rng.randint(5, 50), "fp64", rng.choice(["wcns", "wcns", "four_eq"]),
                    bounds=rng.choice(["open", "periodic"]))
    if kind == "plane":
        n = (size(40, 2048), size(20, 1024))
        wt = rng.choice(["is", "is", "is", "mlp"])
        bounds = "open" if wt == "mlp" else rng.choice(["open", "periodic", "inflow", "mixed"])
        return grid(None, n, sp, rng.randint(1, 5), "fp64" if wt == "mlp" else prec, "wcns", wt, bounds,
                    rng.choice(["advance", "advance", "stages"]))
    if kind == "cube":
        n = (size(20, 230), size(20, 230), size(20, 230))
        return grid(None, n, sp, rng.randint(1, 2), prec, bounds=rng.choice(["open", "periodic", "mixed"]),
                    call=rng.choice(["advance", "advance", "stages"]))
    if kind == "ensemble":
        lo = size(20, 400)
        return ensemble(None, size(50, 4000), lo, lo + size(20, 1500), sp, 10, prec)
    if kind == "train":
        return dict(kind="train", pairs=size(20000, 2000000), batch=size(1000, 65536), steps=rng.randint(2, 8))
    n = (size(100, 4096), size(60, 2048))
    return dict(kind="output", n0=n[0], n1=n[1], n2=1, dim=2, species=sp)


# ---------------------------------------------------------------- inputs
def species_table(case):
    """gamma, c_v, p_inf of the case's species: one liquid, the rest gases."""
    three = case["species"] == 3
    table = [LIQUID_B, AIR, LIGHT] if three else [LIQUID_A, AIR]
    return [t[0] for t in table], [t[1] / t[0] for t in table], [t[2] for t in table]


def mixed_state(eos, alpha, u, p, T):
    """Conservative state of volume fractions (all but the last), velocities, p and T."""
    g, cv, pinf = eos
    last = 1.0 - sum(alpha)
    al = list(alpha) + [last]
    ar = [al[k] * (p + pinf[k]) / ((g[k] - 1.0) * cv[k] * T) for k in range(len(g))]
    rho = sum(ar)
    E = 0.5 * rho * sum(v * v for v in u)
    for k in range(len(g)):
        E = E + al[k] * (p + g[k] * pinf[k]) / (g[k] - 1.0)
    return torch.stack(ar + [rho * v for v in u] + [E] + list(alpha))


def modes(r, coords, count, high):
    """Sum of `count` random cosine modes over the coordinates, at most 1 in size."""
    s = 0.0
    for _ in range(count):
        arg = r.uniform(0.0, 2.0 * math.pi)
        for x, length in coords:
            arg = arg + 2.0 * math.pi * int(r.integers(1, high + 1)) * x / length
        s = s + torch.cos(arg)
    return s / count


def flow(case, seed):
    """State (M, n2, n1, n0) of a shock meeting liquid and gas interfaces; (state, spacing, inflow or None)."""
    r = np.random.default_rng(int(seed))
    D, N, n = case["dim"], case["species"], (case["n0"], case["n1"], case["n2"])
    eos = species_table(case)
    dx = 1.0 / n[0]
    axes = [(torch.arange(n[d], dtype=torch.float64, device="cuda") + 0.5) * dx for d in range(3)]
    shape = (n[2], n[1], n[0])
    X = [axes[0].view(1, 1, -1), axes[1].view(1, -1, 1), axes[2].view(-1, 1, 1)]
    lengths = [n[d] * dx for d in range(3)]
    coords = [(X[d], lengths[d]) for d in range(D)]
    zero = torch.zeros(shape, dtype=torch.float64, device="cuda")
    width = 2.0 * dx
    planar = D == 1 or case.get("weights") == "mlp"
    if planar:
        # liquid at high pressure against air at 1 bar
        at = r.uniform(0.4, 0.7)
        left = (X[0] < at).to(torch.float64) + zero
        high = math.exp(r.uniform(math.log(1e8), math.log(1e9)))
        p = left * high * (1.0 + 0.05 * modes(r, coords[:1], 2, 4)) + (1.0 - left) * 1e5
        rho_l, rho_r = r.uniform(900.0, 1100.0), r.uniform(20.0, 60.0)
        g, cv, pinf = eos
        T = left * (high + pinf[0]) / ((g[0] - 1.0) * rho_l * cv[0]) + (1.0 - left) * 1e5 / ((g[1] - 1.0) * rho_r * cv[1])
        alpha = [TRACE + (1.0 - 3.0 * TRACE) * left]
        if N == 3:
            alpha.append(TRACE + (1.0 - 3.0 * TRACE) * (1.0 - left) * (X[0] < 0.5 * (1.0 + at)))
        u = [5.0 * modes(r, coords, 2, 4) + zero for _ in range(D)]
        return mixed_state(eos, alpha, u, p, T), dx, None
    # liquid drops in gas, a perturbed gas interface (three species), a Mach-1.47 shock in air behind them
    liquid = zero.clone()
    for _ in range(10 if D == 2 else 24):
        centre = [r.uniform(0.4, 0.95)] + [r.uniform(0.0, lengths[d]) for d in range(1, D)]
        rad = r.uniform(0.02, 0.08)
        d2 = sum((X[d] - centre[d]) ** 2 for d in range(D))
        liquid = torch.maximum(liquid, 0.5 * (1.0 - torch.tanh((torch.sqrt(d2) - rad) / width)))
    if case.get("bounds") == "periodic":  # no shock: smooth pressure and velocity everywhere
        post = zero
    else:
        post = (X[0] < r.uniform(0.15, 0.3)).to(torch.float64) + zero
    ga, cva = eos[0][1], eos[1][1]
    m2, c0 = 1.47 ** 2, math.sqrt(1.4 * 0.4 * cva * T0)
    p1 = P0 * (1.0 + 2.0 * ga / (ga + 1.0) * (m2 - 1.0))
    jump = (ga + 1.0) * m2 / ((ga - 1.0) * m2 + 2.0)
    u1 = 1.47 * c0 * (1.0 - 1.0 / jump)
    p = (P0 + (p1 - P0) * post) * (1.0 + 0.01 * modes(r, coords, 3, 6))
    T = T0 + T0 * (p1 / P0 / jump - 1.0) * post + zero
    u = [5.0 * modes(r, coords, 3, 6) + zero for _ in range(D)]
    u[0] = u[0] + u1 * post
    alpha = [TRACE + (1.0 - 3.0 * TRACE) * liquid]
    if N == 3:
        wavy = X[0] - 0.5 - 0.02 * (modes(r, coords[1:], 4, 8) if D > 1 else 0.0)
        air = 0.5 * (1.0 - torch.tanh(wavy / width))
        alpha.append(TRACE + (1.0 - 3.0 * TRACE) * (1.0 - liquid) * air)
    inflow = None
    if case.get("bounds") == "inflow":
        y = X[1].view(-1)
        jet = ((y - 0.5 * lengths[1]).abs() <= 0.1 * lengths[1]).to(torch.float64)
        a = [TRACE + (1.0 - 3.0 * TRACE) * jet] + [TRACE + (1.0 - 3.0 * TRACE) * (1.0 - jet)] * (N - 2)
        inflow = mixed_state(eos, a, [300.0 * jet] + [torch.zeros_like(y)] * (D - 1), P0 + 0.0 * y, T0 + 0.0 * y).contiguous()
    return mixed_state(eos, alpha, u, p, T), dx, inflow


def tubes(case, seed):
    """Shock tubes back to back: liquid at 1e7 to 1e9 Pa or gas against gas at 1e5 to 1e6 Pa, on either side (a
    liquid pulled into tension would make the common pressure ill-conditioned): (state (M, cells), offsets, spacing
    per problem)."""
    r = np.random.default_rng(int(seed))
    N, B = case["species"], case["problems"]
    eos = species_table(case)
    # the lengths belong to the case, not to the seed: a pass is the same work for every seed
    lens = np.random.default_rng(77).integers(case["shortest"], case["longest"] + 1, size=B)
    off = np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)

    def dev(a):
        return torch.from_numpy(np.ascontiguousarray(a)).cuda()

    sides = []
    liquid_at = r.integers(-1, 2, B)  # the side that is liquid, -1: neither
    for side in range(2):
        major = np.where(liquid_at == side, 0, r.integers(1, N, B))
        p = np.exp(r.uniform(0.0, 1.0, B) * np.where(major == 0, math.log(1e2), math.log(1e1))) * np.where(major == 0, 1e7, 1e5)
        rho = np.where(major == 0, r.uniform(800.0, 1200.0, B), np.exp(r.uniform(0.0, math.log(50.0), B)))
        g, cv, pinf = (np.asarray(t)[major] for t in eos)
        al = np.where(np.arange(N)[:, None] == major, 1.0 - (N - 1) * TRACE, TRACE)
        sides.append((p, (p + pinf) / ((g - 1.0) * rho * cv), al))
    b = torch.repeat_interleave(torch.arange(B, device="cuda"), dev(lens))
    i = torch.arange(int(off[-1]), device="cuda") - dev(off)[b]
    left = (i.to(torch.float64) + 0.5) < 0.5 * dev(lens)[b].to(torch.float64)
    pick = [torch.where(left, dev(x)[..., b], dev(y)[..., b]) for x, y in zip(*sides)]
    u = [torch.zeros_like(pick[0])]
    return mixed_state(eos, [pick[2][k] for k in range(N - 1)], u, pick[0], pick[1]), off, 1.0 / lens


def stencils(case, seed):
    """Normalised training pairs of the kinds the extraction gives: smooth profiles and jumps."""
    g = torch.Generator(device="cuda").manual_seed(int(seed))
    n = case["pairs"]

    def rnd(*s):
        return torch.rand(*s, generator=g, device="cuda", dtype=torch.float64)

    j = torch.arange(-2, 3, device="cuda", dtype=torch.float64)
    k, ph, at = 0.1 + 1.5 * rnd(n, 1), 6.3 * rnd(n, 1), 4.0 * rnd(n, 1) - 2.0
    step = (rnd(n, 1) < 0.3).to(torch.float64) * (4.0 * rnd(n, 1) - 2.0)

    def value(x):
        return torch.sin(k * x + ph) + step * torch.tanh((x - at) / 0.2)

    u, label = value(j), value(0.5 + 0.0 * j[:1])
    d = u - u[:, 2:3]
    s = 1.0 / d.abs().amax(1, keepdim=True).clamp_min(1e-12)
    t = (label - u[:, 2:3]) * s
    X = torch.zeros(n, 8, device="cuda", dtype=torch.float32)
    X[:, :5] = (d * s).to(torch.float32)
    return X, t.view(-1).to(torch.float32)


def optimiser(case, seed):
    """Parameters and Adam moments as they stand in the middle of a training."""
    r = np.random.default_rng(int(seed) + 1)
    p = learned.init_params(int(seed) % 1000, last_scale=0.5)
    m = (1e-3 * r.standard_normal(p.size)).astype(np.float32)
    v = (1e-5 * (0.5 + r.uniform(size=p.size))).astype(np.float32)
    return [torch.from_numpy(a).cuda() for a in (p, m, v)]


def network(seed):
    return learned.init_params(int(seed) % 1000, last_scale=0.5)


def bounds_of(case):
    b = {"open": [(OPEN, OPEN)] * 3, "periodic": [(PERIODIC, PERIODIC)] * 3,
         "mixed": [(OPEN, OPEN), (PERIODIC, PERIODIC), (PERIODIC, PERIODIC)],
         "inflow": [(INFLOW, OPEN), (OPEN, OPEN), (OPEN, OPEN)]}[case.get("bounds", "open")]
    if case.get("weights") == "mlp" and case["bounds"] == "open":
        b = [(OPEN, OPEN), (PERIODIC, PERIODIC), (PERIODIC, PERIODIC)]  # planar
    return b


def flags_of(case):
    return hrm.FUSE_RELAX | (hrm.FOUR_EQ if case.get("scheme") == "four_eq" else 0)


# ---------------------------------------------------------------- the library's side
class State:
    """What the program keeps: a handle of the library and device tensors."""

    def __init__(self, case):
        self.case, self.ctx, self.batch = case, 0, 0

    def close(self):
        if self.ctx:
            hrm.hrm_destroy(self.ctx)
        if self.batch:
            hrm.hrm_batch_destroy(self.batch)
        self.ctx = self.batch = 0

    def __del__(self):
        try:
            self.close()
        except Exception:  # the interpreter is ending
            pass


def prepare(case, seed):
    s = State(case)
    if case["kind"] == "train":
        s.X, s.T = stencils(case, seed)
        s.start = optimiser(case, seed)
        s.p, s.m, s.v = (t.clone() for t in s.start)
        s.g, s.loss = torch.zeros_like(s.p), torch.zeros(1, device="cuda")
        s.batch_size = min(case["batch"], case["pairs"])
        s.work = torch.zeros(hrm.hrm_mlp_grad_workspace(s.batch_size), device="cuda")
        return s
    g, cv, pinf = species_table(case)
    eos = hrm.make_eos(g, cv, pinf, [0.0] * len(g))
    prec = hrm.FP32 if case.get("precision") == "fp32" else hrm.FP64
    if case["kind"] == "ensemble":
        s.W0, off, dx = tubes(case, seed)
        s.batch = hrm.hrm_batch_create(eos, None, off, dx, prec)
        s.W = s.W0.clone()
        return s
    W, dx, inflow = flow(case, seed)
    s.W0 = W.contiguous()
    D = case["dim"]
    mlp = case.get("weights") == "mlp"
    spec = hrm.make_grid(D, (case["n0"], case["n1"], case["n2"])[:D], (dx,) * D, bounds_of(case), precision=prec,
                         weights=hrm.WEIGHTS_MLP if mlp else hrm.WEIGHTS_IS, flags=flags_of(case))
    s.ctx = hrm.hrm_create(spec, eos)
    if mlp:
        hrm.hrm_set_mlp(s.ctx, network(seed))
    if inflow is not None:
        s.inflow = inflow
        hrm.hrm_set_boundary_state(s.ctx, 0, 0, inflow)
    s.W = s.W0.clone()
    s.slot = torch.zeros(8, dtype=torch.float64, device="cuda")
    s.maxs = torch.zeros(4, dtype=torch.float64, device="cuda")
    if case.get("call") == "stages":
        s.A, s.B = torch.empty_like(W), torch.empty_like(W)
    if case["kind"] == "output":
        s.out = [torch.empty(W.shape[1:], dtype=torch.float64, device="cuda") for _ in range(3)]
    return s


def run(s):
    c = s.case
    if c["kind"] == "train":
        for t, t0 in zip((s.p, s.m, s.v), s.start):
            t.copy_(t0)
        n = c["pairs"]
        stride = max(1, n // s.batch_size)
        for it in range(c["steps"]):
            hrm.hrm_mlp_grad(s.p, s.X, s.T, (it * 7919) % n, stride, s.batch_size, s.g, s.loss, s.work)
            hrm.hrm_mlp_adam(s.p, s.g, s.m, s.v, 500 + it, 1e-3)
        return {"params": s.p, "grad": s.g, "loss": s.loss}
    s.W.copy_(s.W0)
    if c["kind"] == "ensemble":
        hrm.hrm_batch_run(s.batch, s.W, c["steps"], CFL)
        return parts(s.W, c["species"], 1)
    if c["kind"] == "output":
        hrm.hrm_relax(s.ctx, s.W)
        hrm.hrm_equilibrium_state(s.ctx, s.W, *s.out)
        hrm.hrm_max_wavespeed(s.ctx, s.W, s.maxs)
        return dict(parts(s.W, c["species"], c["dim"]), p=s.out[0], T=s.out[1], c=s.out[2], speeds=s.maxs[:c["dim"]])
    s.slot.zero_()
    if c["call"] == "advance":
        hrm.hrm_advance(s.ctx, s.W, c["steps"], CFL, 0.0, 0.0, s.slot)
    else:
        for _ in range(c["steps"]):
            hrm.hrm_max_wavespeed(s.ctx, s.W, s.maxs)
            hrm.hrm_compute_dt(s.ctx, s.maxs, CFL, 0.0, 0.0, s.slot)
            hrm.hrm_rk_stage(s.ctx, 0, s.W, s.W, s.A, s.slot)
            hrm.hrm_rk_stage(s.ctx, 1, s.W, s.A, s.B, s.slot)
            hrm.hrm_rk_stage(s.ctx, 2, s.W, s.B, s.W, s.slot)
    return dict(parts(s.W, c["species"], c["dim"]), slot=s.slot[:5])


def parts(W, N, D):
    return {"ar": W[:N], "mom": W[N:N + D], "E": W[N + D], "alpha": W[N + D + 1:]}


# ---------------------------------------------------------------- what a pass cannot do without
def face_operations(N, D):
    """One midpoint: 2M interpolations, the flux of the interpolated pair, limiter checks, reconstruction."""
    M = 2 * N + D
    return 253 * M + 141 * N + 56 * D + 251


def step_work(N, D, cells, faces):
    """One three-stage step: each stage reads its state (and W^n after the first) and writes the next."""
    M = 2 * N + D
    cell = D * (8 * N + 3 * D + 7) + D * 2 * M + 4 * M + 12 * N + 2 * D + 25
    return 64 * M * cells, 3 * (faces * face_operations(N, D) + cells * cell)


def work(case):
    if case["kind"] == "train":
        b = min(case["batch"], case["pairs"])
        one = 2 * (5 * 32 + 32 * 32 + 32 * 3)
        return {"bytes": case["steps"] * (b * 24 + 7 * 4 * 1347), "flops": case["steps"] * b * 3 * one}
    N = case["species"]
    if case["kind"] == "ensemble":
        lens = np.random.default_rng(77).integers(case["shortest"], case["longest"] + 1, size=case["problems"])
        cells = int(lens.sum())
        b, f = step_work(N, 1, cells, cells + len(lens))
        return {"bytes": case["steps"] * b, "flops": case["steps"] * f}
    D, n = case["dim"], (case["n0"], case["n1"], case["n2"])
    cells = n[0] * n[1] * n[2]
    if case["kind"] == "output":
        M = 2 * N + D
        return {"bytes": cells * 8 * (2 * M + 3), "flops": cells * 120}
    faces = sum(cells // n[d] * (n[d] + 1) for d in range(D))
    b, f = step_work(N, D, cells, faces)
    if case["scheme"] == "four_eq":
        f = 3 * (faces * 260 + cells * 120)
    return {"bytes": case["steps"] * b, "flops": case["steps"] * f}


# ---------------------------------------------------------------- the same in plain float64 torch
def exact(case, seed):
    if case["kind"] == "train":
        return exact_train(case, seed)
    eos = species_table(case)
    N = case["species"]
    if case["kind"] == "ensemble":
        W, off, dx = tubes(case, seed)
        if W.shape[1] * case["steps"] > 60e6:
            return None
        return parts(exact_ensemble(eos, W, off, dx, case["steps"]), N, 1)
    D = case["dim"]
    W, dx, inflow = flow(case, seed)
    if case["kind"] == "output":
        W = relax(eos, W, D)
        p, T, c = equilibrium(eos, W, D)
        speeds = torch.stack([s.max() for s in speeds_of(eos, W, D, False)])
        return dict(parts(W, N, D), p=p, T=T, c=c, speeds=speeds)
    if W[0].numel() * case["steps"] * D > 110e6:
        return None
    four = case["scheme"] == "four_eq"
    net = network(seed) if case["weights"] == "mlp" else None
    t = 0.0
    for _ in range(case["steps"]):
        top = [s.max() for s in speeds_of(eos, W, D, four)]
        if inflow is not None:
            top[0] = torch.maximum(top[0], speeds_of(eos, inflow, D, four)[0].max())
        tau = [m / dx for m in top]
        dt = CFL / sum(tau)
        lam = [dt / (ta / sum(tau) * dx) for ta in tau]
        Wn = W
        for a, b in ((0.0, 1.0), (0.75, 0.25), (1.0 / 3.0, 2.0 / 3.0)):
            L = 0.0
            for d in range(D):
                L = L + line_rhs(eos, W, D, d, bounds_of(case)[d], inflow if d == 0 else None, lam[d], dx, four, net)
            W = relax(eos, a * Wn + b * (W + dt * L), D)
        t = t + dt
    slot = torch.stack([dt] + lam + [torch.zeros_like(dt)] * (3 - D) + [t])
    return dict(parts(W, N, D), slot=slot)


def line_rhs(eos, W, D, d, bc, inflow, lam, dx, four, net):
    """-(G^-_{i+1/2} - G^+_{i-1/2}) / dx along direction d, in slabs of lines."""
    N, M = len(eos[0]), W.shape[0]
    V = W.movedim(3 - d, -1)
    n, lines = V.shape[-1], V.shape[1:-1]
    V = V.reshape(M, -1, n)
    out = torch.empty_like(V)
    per = max(1, int(1e6) // (n + 1))
    for l0 in range(0, V.shape[1], per):
        v = V[:, l0:l0 + per]
        if bc[0] == PERIODIC:
            v = torch.cat([v[..., -3:], v, v[..., :3]], -1)
        else:
            lo = v[..., :1] if inflow is None else inflow.reshape(M, -1, 1)[:, l0:l0 + per]
            v = torch.cat([lo.expand(-1, -1, 3), v, v[..., -1:].expand(-1, -1, 3)], -1)
        nodes = [v[..., j:j + n + 1] for j in range(6)]
        G, Gp = face(eos, nodes, D, d, lam, four, net)
        plus = torch.cat([G[:N + D + 1], Gp])
        out[:, l0:l0 + per] = -(G[..., 1:] - plus[..., :-1]) / dx
    return out.reshape((M,) + lines + (n,)).movedim(-1, 3 - d)


def exact_ensemble(eos, W, off, dx, steps):
    lens = np.diff(off)
    B = len(lens)
    cell_b = torch.repeat_interleave(torch.arange(B), torch.from_numpy(lens)).cuda()
    face_b = torch.repeat_interleave(torch.arange(B), torch.from_numpy(lens + 1)).cuda()
    start = torch.from_numpy(off[:-1]).cuda()
    end = torch.from_numpy(off[1:]).cuda()
    dxs = torch.from_numpy(np.asarray(dx)).cuda()
    f = torch.arange(face_b.numel(), device="cuda") - face_b  # cell to the right of the face
    nodes_at = [torch.minimum(torch.maximum(f - 3 + j, start[face_b]), end[face_b] - 1) for j in range(6)]
    left = torch.arange(cell_b.numel(), device="cuda") + cell_b
    N = len(eos[0])
    for _ in range(steps):
        sp = speeds_of(eos, W, 1, False)[0]
        top = torch.zeros(B, dtype=torch.float64, device="cuda").scatter_reduce(0, cell_b, sp, "amax")
        dt = CFL / (top / dxs)
        lam = dt / dxs
        Wn = W
        for a, b in ((0.0, 1.0), (0.75, 0.25), (1.0 / 3.0, 2.0 / 3.0)):
            L = torch.empty_like(W)
            G, Gp = (torch.empty(k, f.numel(), dtype=torch.float64, device="cuda") for k in (W.shape[0], N - 1))
            for c0 in range(0, f.numel(), 1 << 20):
                c1 = min(c0 + (1 << 20), f.numel())
                G[:, c0:c1], Gp[:, c0:c1] = face(eos, [W[:, i[c0:c1]] for i in nodes_at], 1, 0, lam[face_b[c0:c1]],
                                                 False, None)
            plus = torch.cat([G[:N + 2], Gp])
            L = -(G[:, left + 1] - plus[:, left]) / dxs[cell_b]
            W = relax(eos, a * Wn + b * (W + dt[cell_b] * L), 1)
    return W


def primitive(eos, W, D):
    """Partial densities, velocities, p, all volume fractions, rho, c, rho c^2, E of a conservative state."""
    g, cv, pinf = eos
    N = len(g)
    ar, mom, E = list(W[:N]), list(W[N:N + D]), W[N + D]
    al = list(W[N + D + 1:])
    al.append(1.0 - sum(al))
    rho = sum(ar)
    Gam = sum(al[k] / (g[k] - 1.0) for k in range(N))
    Pi = sum(al[k] * g[k] * pinf[k] / (g[k] - 1.0) for k in range(N))
    u = [m / rho for m in mom]
    p = (E - 0.5 * sum(m * m for m in mom) / rho - Pi) / Gam
    rc2 = p + (p + Pi) / Gam
    return dict(ar=ar, u=u, p=p, al=al, rho=rho, c=torch.sqrt(rc2 / rho), rc2=rc2, E=E, mom=mom)


def complete(eos, V):
    """The rest of a state from partial densities, velocities, p and volume fractions."""
    g, cv, pinf = eos
    N = len(g)
    al = list(V["al"][:N - 1])
    al.append(1.0 - sum(al))
    rho = sum(V["ar"])
    Gam = sum(al[k] / (g[k] - 1.0) for k in range(N))
    Pi = sum(al[k] * g[k] * pinf[k] / (g[k] - 1.0) for k in range(N))
    p = V["p"]
    rc2 = p + (p + Pi) / Gam
    E = Gam * p + Pi + 0.5 * rho * sum(v * v for v in V["u"])
    return dict(V, al=al, rho=rho, rc2=rc2, c=torch.sqrt(rc2 / rho), E=E, mom=[rho * v for v in V["u"]])


def weno(v, net):
    """Value at i+1/2 from nodes i-2..i+2."""
    a, b, c, d, e = v
    if net is not None:
        return learned_value(v, net)
    cand = (0.5 * (c + d), 0.5 * (3 * c - b), (3 * c + 6 * d - e) / 8, (3 * a - 10 * b + 15 * c) / 8)
    k = 13.0 / 12.0
    b0, b1 = (c - d) ** 2, (b - c) ** 2
    b01 = k * (b - 2 * c + d) ** 2 + 0.25 * (b - d) ** 2
    b2 = k * (c - 2 * d + e) ** 2 + 0.25 * (3 * c - 4 * d + e) ** 2
    b3 = k * (a - 2 * b + c) ** 2 + 0.25 * (a - 4 * b + 3 * c) ** 2
    t = k * (e - 4 * d + 6 * c - 4 * b + a) ** 2 + 0.25 * (e - 2 * d + 2 * b - a) ** 2
    B0, B1, B01, B2, B3 = (x + 1e-15 for x in (b0, b1, b01, b2, b3))
    w = (15.0 / 32.0 * (1 + t * t / (B0 * B01)), 5.0 / 32.0 * (1 + t * t / (B1 * B01)), 5.0 / 16.0 * (1 + t / B2),
         1.0 / 16.0 * (1 + t / B3))
    return sum(x * s for x, s in zip(w, cand)) / sum(w)


def learned_value(v, P):
    P = torch.from_numpy(P.astype(np.float64)).cuda()
    u = torch.stack(list(v), -1)
    shape = u.shape[:-1]
    u = u.reshape(-1, 5)
    d = u - u[:, 2:3]
    s = d.abs().amax(1, keepdim=True)
    x = d * torch.where(s > 0, 1.0 / s, torch.zeros_like(s))
    w = omega(x, P)[0]
    sl, sc, sr = candidates(u)
    return (sc + w[:, 0] * (sl - sc) + w[:, 2] * (sr - sc)).reshape(shape)


def candidates(u):
    return ((3 * u[:, 0] - 10 * u[:, 1] + 15 * u[:, 2]) / 8, (-u[:, 1] + 6 * u[:, 2] + 3 * u[:, 3]) / 8,
            (3 * u[:, 2] + 6 * u[:, 3] - u[:, 4]) / 8)


def omega(x, P):
    h = torch.relu(x @ P[:160].view(5, 32) + P[160:192])
    h = torch.relu(h @ P[192:1216].view(32, 32) + P[1216:1248])
    z = h @ P[1248:1344].view(32, 3) + P[1344:1347]
    a, b, c, d, e = (x[:, j] for j in range(5))
    k = 13.0 / 12.0
    beta = torch.stack([k * (a - 2 * b + c) ** 2 + 0.25 * (a - 4 * b + 3 * c) ** 2,
                        k * (b - 2 * c + d) ** 2 + 0.25 * (b - d) ** 2,
                        k * (c - 2 * d + e) ** 2 + 0.25 * (3 * c - 4 * d + e) ** 2], 1)
    lin = torch.tensor([1.0 / 16.0, 10.0 / 16.0, 5.0 / 16.0], dtype=torch.float64, device="cuda")
    w = lin * torch.exp(torch.tanh(z)) / (1e-6 + beta) ** 2
    return w / w.sum(1, keepdim=True), z


def limited(eos, V, node):
    """Interpolation limiter: blend partial densities and volume fractions, then the hard switch."""
    N = len(eos[0])
    ar = []
    for k in range(N):
        a, b = node["ar"][k], V["ar"][k]
        m = a.clamp_max(1e-10)
        ar.append(torch.where(b < m, m, b))
    at = list(V["al"][:N - 1])
    at.append(1.0 - sum(at))
    th = torch.ones_like(ar[0])
    for k in range(N):
        th = torch.minimum(th, theta(node["al"][k], at[k], 1e-10))
    al = [torch.where(th < 1.0, (1 - th) * node["al"][k] + th * at[k], at[k]) for k in range(N - 1)]
    V = complete(eos, dict(V, ar=ar, al=al))
    bad = ~torch.isfinite(V["rc2"]) | ~torch.isfinite(V["p"]) | (V["rc2"] < node["rc2"].clamp_max(1e-9))
    for k in range(N):
        bad |= (V["ar"][k] < node["ar"][k].clamp_max(1e-11)) | (V["al"][k] < node["al"][k].clamp_max(1e-11))
    if bool(bad.any()):
        V = {k: [torch.where(bad, y, x) for x, y in zip(V[k], node[k])] if isinstance(V[k], list)
             else torch.where(bad, node[k], V[k]) for k in V}
    return V


def theta(a, b, eps):
    m = a.clamp_max(eps)
    return torch.where(b < m, (a - m) / (a - b), torch.ones_like(a))


def star_flux(L, R, d, pc=None):
    """HLLC flux (five-equation, or with the given pressures and sound speeds) and the contact speed."""
    pL, cL, pR, cR = pc if pc else (L["p"], L["c"], R["p"], R["c"])
    uL, uR = L["u"][d], R["u"][d]
    ub, cb = 0.5 * (uL + uR), 0.5 * (cL + cR)
    sL, sR = torch.minimum(ub - cb, uL - cL), torch.maximum(ub + cb, uR + cR)
    ss = (pR - pL + L["rho"] * uL * (sL - uL) - R["rho"] * uR * (sR - uR)) / (L["rho"] * (sL - uL) - R["rho"] * (sR - uR))
    wl = 0.5 * (1.0 + torch.sign(ss))
    sides = []
    for S, p, sk, cap in ((L, pL, sL, sL.clamp_max(0.0)), (R, pR, sR, sR.clamp_min(0.0))):
        u = S["u"][d]
        chi = (sk - u) / (sk - ss)
        f = [a * u + cap * (chi * a - a) for a in S["ar"]]
        for q, m in enumerate(S["mom"]):
            star = chi * S["rho"] * (ss if q == d else S["u"][q])
            f.append(m * u + (p if q == d else 0.0) + cap * (star - m))
        Es = chi * (S["E"] + (ss - u) * (S["rho"] * ss + p / (sk - u)))
        f.append((S["E"] + p) * u + cap * (Es - S["E"]))
        f += [a * ss for a in S["al"][:-1]]
        sides.append(torch.stack(f))
    return wl * sides[0] + (1.0 - wl) * sides[1], ss


def with_alpha(F, L, R, s, N):
    """The pair G^-, G^+ (volume-fraction slots) of a flux F and face velocity s."""
    k = F.shape[0] - (N - 1)
    aL, aR = torch.stack(L["al"][:N - 1]), torch.stack(R["al"][:N - 1])
    return torch.cat([F[:k], F[k:] - s * aL]), F[k:] - s * aR


def face(eos, W6, D, d, lam, four, net):
    N = len(eos[0])
    q = [primitive(eos, w, D) for w in W6]
    L, R = q[2], q[3]
    if four:
        pL, _, cL = equilibrium(eos, W6[2], D)
        pR, _, cR = equilibrium(eos, W6[3], D)
        F, _ = star_flux(L, R, d, (pL, cL, pR, cR))
        F[N + D + 1:] = 0.0
        return F, torch.zeros_like(F[N + D + 1:])
    F1, s1 = star_flux(L, R, d)
    lo, lo_p = with_alpha(F1, L, R, s1, N)
    arb = [0.5 * (L["ar"][k] + R["ar"][k]) for k in range(N)]
    rb, cb = 0.5 * (L["rho"] + R["rho"]), 0.5 * (L["c"] + R["c"])

    def both(f):
        v = [f(x) for x in q]
        return weno(v[:5], net), weno(v[:0:-1], net)

    first = both(lambda x: x["u"][d] - x["p"] / (rb * cb))
    last = both(lambda x: x["u"][d] + x["p"] / (rb * cb))
    mid = [both(lambda x, k=k: x["ar"][k] - arb[k] / (rb * cb * cb) * x["p"]) for k in range(N)]
    cross = {e: both(lambda x, e=e: x["u"][e]) for e in range(D) if e != d}
    al = [both(lambda x, k=k: x["al"][k]) for k in range(N - 1)]
    V = []
    for s, node in ((0, L), (1, R)):
        du = last[s] - first[s]
        v = dict(ar=[mid[k][s] + arb[k] * 0.5 / cb * du for k in range(N)], p=0.5 * rb * cb * du,
                 u=[0.5 * (first[s] + last[s]) if e == d else cross[e][s] for e in range(D)],
                 al=[al[k][s] for k in range(N - 1)])
        V.append(limited(eos, v, node))
    Gt, ut = star_flux(V[0], V[1], d)

    def ratio(f):
        a = [f(x) for x in q]
        r = []
        for o in (0, 1):
            w = a[o:o + 5]
            num = (-w[0] + 16 * w[1] - 30 * w[2] + 16 * w[3] - w[4]).abs()
            den = (w[0] + 16 * w[1] + 30 * w[2] + 16 * w[3] + w[4]).abs()
            r.append(torch.where(den > 0, num / den, (num > 0).to(num.dtype)))
        return 0.5 * (r[0] + r[1])

    z = ratio(lambda x: x["rho"]) * ratio(lambda x: x["p"])
    sig = torch.tanh(1e12 * z * z)
    psi = 256.0 / 175.0
    ca, cb_, cc = 75.0 * psi / 128.0 - 37.0 / 60.0, 25.0 * psi / 256.0 - 2.0 / 15.0, 3.0 * psi / 256.0 - 1.0 / 60.0

    def blend(t, g):
        h = psi * t - ca * (g[2] + g[3]) + cb_ * (g[1] + g[4]) - cc * (g[0] + g[5])
        return sig * t + (1.0 - sig) * h

    flux = [node_flux(x, w, D, d, True) for x, w in zip(q, W6)]
    G = blend(Gt, flux)
    uh = blend(ut, [x["u"][d] for x in q])
    hi, hi_p = with_alpha(G, L, R, uh, N)
    return flux_limited(eos, D, W6[2], W6[3], node_flux(L, W6[2], D, d, False), node_flux(R, W6[3], D, d, False),
                        lam, hi, hi_p, lo, lo_p)


def node_flux(x, W, D, d, alpha):
    """Flux of a node state; the volume-fraction slots hold u alpha, or 0 in the quasi-conservative form."""
    N = len(x["ar"])
    f = W * x["u"][d]
    f[N + d] += x["p"]
    f[N + D] += x["p"] * x["u"][d]
    if not alpha:
        f[N + D + 1:] = 0.0
    return f


def flux_limited(eos, D, WL, WR, FL, FR, lam, hi, hi_p, lo, lo_p):
    N = len(eos[0])
    k = N + D + 1

    def halves(G, Gp):
        return WL - 2 * lam * (G - FL), WR + 2 * lam * (torch.cat([G[:k], Gp]) - FR)

    def alphas(W):
        a = list(W[k:])
        return a + [1.0 - sum(a)]

    def energy(W):
        return W[N + D] - 0.5 * (W[N:N + D] ** 2).sum(0) / W[:N].sum(0)

    low, high = halves(lo, lo_p), halves(hi, hi_p)
    th = torch.ones_like(WL[0])
    for a, b in zip(low, high):
        for j in range(N):
            th = torch.minimum(th, theta(a[j], b[j], 1e-10))
        for x, y in zip(alphas(a), alphas(b)):
            th = torch.minimum(th, theta(x, y, 1e-10))
    G, Gp = (1 - th) * lo + th * hi, (1 - th) * lo_p + th * hi_p
    th = torch.ones_like(th)
    for a, b in zip(low, halves(G, Gp)):
        th = torch.minimum(th, theta(energy(a), energy(b), 1e-8))
    G, Gp = (1 - th) * lo + th * G, (1 - th) * lo_p + th * Gp
    bad = ~torch.isfinite(G).all(0)
    for a, b in zip(low, halves(G, Gp)):
        for j in range(N):
            bad |= b[j] < a[j].clamp_max(1e-11)
        for x, y in zip(alphas(a), alphas(b)):
            bad |= y < x.clamp_max(1e-11)
        e = energy(b)
        bad |= ~torch.isfinite(e) | (e < energy(a).clamp_max(1e-9))
    return torch.where(bad, lo, G), torch.where(bad, lo_p, Gp)


def relaxed(eos, W, D):
    """Common p and T of the species, and where they exist."""
    g, cv, pinf = eos
    N = len(g)
    rho = W[:N].sum(0)
    Y = [W[k] / rho for k in range(N)]
    cvb, cpb = sum(y * c for y, c in zip(Y, cv)), sum(y * a * c for y, a, c in zip(Y, g, cv))
    re = W[N + D] - 0.5 * (W[N:N + D] ** 2).sum(0) / rho
    p1, R1 = pinf[0], g[0] * cv[0] - cv[0]
    B = -(re * (cpb - cvb) - p1 * cvb - p1 * Y[0] * R1)
    C = -re * p1 * ((cpb - cvb) - Y[0] * R1)
    root = torch.sqrt(B * B - 4.0 * cvb * C)
    p = torch.where(B <= 0, (-B + root) / (2.0 * cvb), 2.0 * C / (-B - root))
    T = re / rho / (Y[0] * (p + g[0] * p1) * cv[0] / (p + p1) + cvb - Y[0] * cv[0])
    return p, T, (re > 0) & (rho > 0) & (p > 0) & (T > 0) & torch.isfinite(p) & torch.isfinite(T)


def relax(eos, W, D):
    g, cv, pinf = eos
    N = len(g)
    p, T, ok = relaxed(eos, W, D)
    W = W.clone()
    for k in range(N - 1):
        W[N + D + 1 + k] = torch.where(ok, W[k] * (g[k] - 1.0) * cv[k] * T / (p + pinf[k]), W[N + D + 1 + k])
    return W


def equilibrium(eos, W, D):
    """p, T and the sound speed of the four-equation model."""
    g, cv, pinf = eos
    N = len(g)
    p, T, ok = relaxed(eos, W, D)
    m = W[:N]
    rho = m.sum(0)
    re = W[N + D] - 0.5 * (W[N:N + D] ** 2).sum(0) / rho
    Sv = sum(m[k] * cv[k] for k in range(N))
    SR = sum(m[k] * (g[k] - 1.0) * cv[k] for k in range(N))
    S2 = SR - m[0] * (g[0] - 1.0) * cv[0]
    c = torch.sqrt(p * (re + p) * (SR * p + pinf[0] * S2) / (rho * (Sv * p * p + re * pinf[0] * S2)))
    nan = torch.full_like(p, math.nan)
    return torch.where(ok, p, nan), torch.where(ok, T, nan), torch.where(ok, c, nan)


def speeds_of(eos, W, D, four):
    x = primitive(eos, W, D)
    c = equilibrium(eos, W, D)[2] if four else x["c"]
    return [v.abs() + c for v in x["u"]]


def exact_train(case, seed):
    X, T = stencils(case, seed)
    p, m, v = (t.to(torch.float64) for t in optimiser(case, seed))
    n, b = case["pairs"], min(case["batch"], case["pairs"])
    stride = max(1, n // b) % n or 1
    for it in range(case["steps"]):
        at = ((it * 7919) % n + torch.arange(b, device="cuda") * stride) % n
        x, t = X[at, :5].to(torch.float64), T[at].to(torch.float64)
        q = p.clone().requires_grad_(True)
        w = omega(x, q)[0]
        loss = ((w * torch.stack(candidates(x), 1)).sum(1) - t).square().mean()
        grad = torch.autograd.grad(loss, q)[0]
        m, v = 0.9 * m + 0.1 * grad, 0.999 * v + 0.001 * grad * grad
        k = 500 + it
        p = p - 1e-3 * (m / (1 - 0.9 ** k)) / (torch.sqrt(v / (1 - 0.999 ** k)) + 1e-8)
    return {"params": p, "grad": grad, "loss": loss.detach().view(1)}
