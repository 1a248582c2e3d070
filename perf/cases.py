"""The work that users of this framework run, as cases that can be timed and whose outputs can be compared.

A case is a dict of plain values with a "kind":

  step      whole Runge-Kutta steps of one block (asterx.Block), launched eagerly or replayed from a captured HIP
            graph: the main path (recovery, ghost fills, faces, divergence, constrained transport, stage outputs)
  patches   Heun steps of a set of uneven patches advanced together (asterx.Batch)
  gradient  the density loss of a periodic run and its gradient with respect to the initial primitives and the
            adiabatic index (adjoint.py): forward with checkpoints, then reverse
  recover   one recovery with sources (asterx.c2p_src) of a star in a near-vacuum atmosphere: most cells fail or are
            reset, the rest iterate
  points    recovery of independent points (asterx.c2p_points), cold or warm started
  levels    prolongation and restriction of the nine evolved fields between two refinement levels
  train     one training step of the learned guess's network (gradient and Adam)

exact() computes the same results in plain torch, in 64 bits, from the equations: no kernel of the library is used.
Inputs are made on the GPU from the seed.
"""
import math
import random

import numpy as np
import torch

from paper_2406_11669_amd import adjoint
from paper_2406_11669_amd import asterx as ax
from paper_2406_11669_amd import workloads as W

F64 = torch.float64
SIDES = (16, 24, 32, 48)


# ---- the cases ----------------------------------------------------------------------------------------------

def _step(name, n, data, recon, rk, steps, graph, riemann="hlle", ct="fct", speeds="quartic", gauge="lorenz",
          tmunu=False):
    n = (n, n, n) if isinstance(n, int) else n
    c = dict(kind="step", nx=n[0], ny=n[1], nz=n[2], data=data, recon=recon, riemann=riemann, ct=ct, speeds=speeds,
             gauge=gauge, rk=rk, steps=steps, graph=graph, tmunu=tmunu)
    return dict(c, name=name) if name else c


def listed():
    return [
        # the smallest calls: a test-sized Riemann block stepped from Python, bound by launches and latency
        _step("step_riemann16", 16, "riemann", "minmod", 2, 4, False),
        # the Riemann block of the framework's own workloads (32^3, ten Heun steps), replayed from a graph
        _step("step_riemann32_graph", 32, "riemann", "minmod", 2, 10, True),
        # the benchmark: 128^3 in a curved metric, PPM, RK4, replayed from a graph
        _step("step_curved128_ppm", 128, "curved", "ppm", 4, 1, True),
        # the same block with the fifth-order scheme
        _step("step_curved128_wenoz", 128, "curved", "wenoz", 4, 1, True),
        # the cell count of the paper's single-GPU benchmark, launched eagerly
        _step("step_curved240_ppm", 240, "curved", "ppm", 4, 1, False),
        # an odd, ragged block with upwind constrained transport and Lax-Friedrichs fluxes, whose T_mu_nu goes to a
        # spacetime solver after the step
        _step("step_ragged_mp5_uct", (97, 61, 45), "curved", "mp5", 2, 1, False, riemann="lxf", ct="uct", tmunu=True),
        # patches of a refinement hierarchy (a part of the framework's set of 512), persistent launches in a graph
        dict(name="patches_64", kind="patches", patches=64, mix=1, recon="minmod", steps=1, graph=True),
        # differentiation of a run on a 64^3 periodic block (the framework's own size), four steps
        dict(name="gradient_64", kind="gradient", n=64, recon="ppm", rk=2, steps=4),
        # the recovery of a star in vacuum (the paper's single-GPU benchmark spends most of a stage there)
        dict(name="recover_star160", kind="recover", n=160),
        # cold recoveries of independent states, an odd count
        dict(name="points_cold_2000003", kind="points", n=2000003, guess="cold"),
        # refinement boundaries: a 128^3 fine block with its ghosts from a coarse one, and back
        dict(name="levels_128", kind="levels", n=128),
        # one minibatch of the learned guess's training
        dict(name="train_16384", kind="train", n=16384),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["step"] * 5 + ["patches", "gradient", "recover", "points", "points", "levels", "train"])
    if kind == "step":
        data = rng.choice(["riemann", "curved", "curved"])
        ct = rng.choice(["fct", "fct", "fct", "uct"])
        n = tuple(_log_int(rng, 13, 180) for _ in range(3))
        return _step(None, n, data, rng.choice(["minmod", "ppm", "ppm", "wenoz", "mp5"]), rng.choice([2, 4]), 1,
                     rng.random() < 0.5, riemann=rng.choice(["hlle", "hlle", "lxf"]), ct=ct,
                     speeds=rng.choice(["quartic", "quartic", "bound"]),
                     gauge=rng.choice(["lorenz", "lorenz", "algebraic"]), tmunu=rng.random() < 0.2)
    if kind == "patches":
        return dict(kind=kind, patches=_log_int(rng, 3, 80), mix=rng.randrange(1000), recon=rng.choice(["minmod", "ppm", "wenoz"]), steps=1,
                    graph=rng.random() < 0.5)
    if kind == "gradient":
        return dict(kind=kind, n=rng.randint(9, 64), recon=rng.choice(["minmod", "ppm", "ppm"]),
                    rk=rng.choice([2, 4]), steps=rng.randint(1, 3))
    if kind == "recover":
        return dict(kind=kind, n=_log_int(rng, 20, 180))
    if kind == "points":
        return dict(kind=kind, n=_log_int(rng, 500, 4000000), guess=rng.choice(["cold", "warm"]))
    if kind == "levels":
        return dict(kind=kind, n=2 * _log_int(rng, 6, 90))
    return dict(kind=kind, n=_log_int(rng, 64, 60000))


# ---- inputs -------------------------------------------------------------------------------------------------

class Modes:
    """Seeded smooth periodic fields on the unit cube: four low modes each, |f| <= 1."""

    def __init__(self, layout, seed):
        self.L, self.rng = layout, random.Random(seed)

    def __call__(self, where):
        x, y, z = (torch.from_numpy(c).cuda() for c in self.L.coords(where))
        f, norm = 0.0, 0.0
        for _ in range(4):
            k = [0, 0, 0]
            while not any(k):
                k = [self.rng.randint(-2, 2) for _ in range(3)]
            a, ph = self.rng.uniform(0.2, 1.0), self.rng.uniform(0.0, 2.0 * math.pi)
            f = f + a * torch.sin(2.0 * math.pi * (k[0] * x + k[1] * y + k[2] * z) + ph)
            norm += a
        return (f / norm).expand(self.L.shape3)


EDGES = ("xedge", "yedge", "zedge")


def _host(rows):
    return torch.stack(rows).cpu().numpy()


def _curved(case, seed):
    """A periodic block in a curved metric (lapse 0.65 to 0.95, shift to 0.05, metric to 0.1 off flat) with smooth
    fluid, velocity and field, |v| < 0.5, |B| about 1: the distributions of workloads.curved_block."""
    L = W.Layout((case["nx"], case["ny"], case["nz"]), 4 if case["ct"] == "uct" else 3)
    f = Modes(L, seed)
    metric = [0.8 + 0.15 * f("vertex")] + [0.05 * f("vertex") for _ in range(3)]
    metric += [(1.0 if c in (0, 3, 5) else 0.0) + 0.1 * f("vertex") for c in range(6)]
    curv = [0.1 * f("vertex") for _ in range(6)]
    prim = [1.0 + 0.5 * f("centre"), 0.55 + 0.45 * f("centre")] + [0.25 * f("centre") for _ in range(3)]
    A = [0.12 * f(e) for e in EDGES]
    arrays = [L.periodic_wrap(_host(a)) if min(L.n) > 2 * L.ng else _wrap(L, _host(a)) for a in (metric, curv, prim, A)]
    params = W.default_params(gamma=2.0, recon=case["recon"], riemann=case["riemann"], ct=case["ct"],
                              speeds=case["speeds"], gauge=case["gauge"])
    return W.Workload("curved", L, params, *arrays, L.zeros(1), 0.25 * min(L.dx), case["steps"], case["rk"],
                      ("periodic",) * 3, ("periodic",) * 3)


def _wrap(L, a):
    for ax_, d in ((-1, 0), (-2, 1), (-3, 2)):
        a = np.take(a, (np.arange(a.shape[ax_]) - L.ng) % L.n[d] + L.ng, axis=ax_)
    return np.ascontiguousarray(a)


def _step_workload(case, seed):
    if case["data"] == "curved":
        return _curved(case, seed)
    w = W.riemann_block(seed=seed, n=(case["nx"], case["ny"], case["nz"]), ng=4 if case["ct"] == "uct" else 3,
                        recon=case["recon"], rk=case["rk"], nsteps=case["steps"])
    w.params.update(riemann=case["riemann"], ct=case["ct"], speeds=case["speeds"], gauge=case["gauge"])
    return w


def _patches(case, seed):
    """Riemann-problem patches as in workloads.patch_set: uneven sides on three levels (the case's own), one time
    step and one floor for all."""
    mix = random.Random(case["mix"])
    dt, out = 0.25 / 128.0, []
    for q in range(case["patches"]):
        n, dx = mix.choice(SIDES), 2.0 ** -mix.randrange(3) / 32.0
        w = W.riemann_block(seed=seed * 1009 + q, n=n, recon=case["recon"], split=0.5 * n * dx, dx=dx)
        w.dt = dt
        w.params["rho_atm"] = 1e-7
        out.append(w)
    return out


def _graph(step):
    """One captured call of step, after an eager one on a side stream."""
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        step()
    torch.cuda.current_stream().wait_stream(side)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        step()
    return g


def _star(case, seed):
    """A star of 1.4 solar masses (G = c = 1) with a vacuum of floor density around it on [-20, 20]^3, as the cells
    stand between two stages: the star moves slowly; of the vacuum most cells carry a momentum that no state at the
    floor can have, some are below the floor, some are solvable and nearly cold."""
    n = case["n"]
    L = W.Layout((n, n, n), 3, dx=(40.0 / n,) * 3)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    rnd = lambda: torch.rand(L.shape3, generator=gen, dtype=F64, device="cuda")

    def radius(where):
        x, y, z = (torch.from_numpy(c - 20.0).cuda().expand(L.shape3) for c in L.coords(where))
        return x, y, torch.sqrt(x * x + y * y + z * z)

    one, zero = torch.ones(L.shape3, dtype=F64, device="cuda"), torch.zeros(L.shape3, dtype=F64, device="cuda")
    h = 0.7 / torch.sqrt(radius("vertex")[2] ** 2 + 16.0)
    psi4 = (1.0 + h) ** 4
    metric = torch.stack([(1.0 - h) / (1.0 + h), zero, zero, zero, psi4, zero, zero, psi4, zero, psi4])
    curv = torch.zeros((6,) + L.shape3, dtype=F64, device="cuda")
    rho_c, R, floor = 1.28e-3, 8.1, 1.28e-10
    x, y, r = radius("centre")
    q = math.pi * torch.clamp(r / R, 1e-9, 1.0)
    rho = rho_c * torch.sin(q) / q
    inside = (r < R) & (rho > 1e-3 * rho_c)
    rho = torch.where(inside, rho, floor * one)
    p = torch.where(inside, 100.0 * rho ** 2, floor ** 2 * one)
    v = [torch.where(inside, 2e-3 * (2.0 * rnd() - 1.0), zero) for _ in range(3)]
    prim = torch.stack([rho, p] + v)
    A = torch.zeros((3,) + L.shape3, dtype=F64, device="cuda")
    for c, e in ((0, "xedge"), (1, "yedge")):
        xe, ye, re = radius(e)
        f = 2e-7 * torch.clamp(1.0 - (re / (0.8 * R)) ** 2, min=0.0) ** 2
        A[c] = -ye * f if c == 0 else xe * f
    params = W.default_params(gamma=2.0, rho_atm=floor, recon="ppm")
    cons = torch.zeros((5,) + L.shape3, dtype=F64, device="cuda")
    ax.prim2con(L, params, metric, A, prim, cons)
    # the vacuum's conserved variables, well away from the floor and from the bound of physical states
    sg = torch.sqrt(psi4) ** 3
    u, D = rnd(), floor * (1.1 + 0.4 * rnd())
    tau = 1e-8 * D
    low, solvable = u < 0.03, u > 0.8
    D = torch.where(low, 0.8 * D / 1.5, D)
    f = torch.where(solvable, 0.1 + 0.7 * rnd(), 5.0 + 20.0 * rnd())
    S = f * torch.sqrt(tau * (tau + 2.0 * D)) * torch.sqrt(psi4)
    vac = torch.stack([sg * D, sg * S * 0.6, sg * S * 0.48, sg * S * 0.64, sg * tau])
    cons = torch.where(inside, cons, vac)
    return L, params, metric, curv, A, cons, prim


def _points(case, seed):
    """States of the framework's recovery benchmark (rho, p in [0.1, 1], B^i in [-1, 1], W in [1, 10], isotropic
    velocities), in metrics up to 0.1 off flat."""
    n = case["n"]
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    rnd = lambda *s: torch.rand(s + (n,), generator=gen, dtype=F64, device="cuda")
    m = 0.1 * (2.0 * rnd(10) - 1.0)
    m[0] += 0.8
    for c in (4, 7, 9):
        m[c] += 1.0
    g = m[4:]
    d = 2.0 * rnd(3) - 1.0
    lorentz = 1.0 + 9.0 * rnd()
    v = d * torch.sqrt((1.0 - 1.0 / lorentz ** 2) / _dot(d, _lower(g, d)))
    prim = torch.cat([0.1 + 0.9 * rnd(2), v])
    Bt = (2.0 * rnd(3) - 1.0) * torch.sqrt(_det(g))
    cons = torch.stack(_cons(_geo(m), _fluid(_geo(m), prim, Bt, 5.0 / 3.0))).contiguous()
    guess = prim * (1.0 + 1e-3 * (2.0 * rnd(5) - 1.0)) if case["guess"] == "warm" else None
    return m, prim, Bt, cons, guess


def _train_data(case, seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    n = case["n"]
    feat = torch.randn((8, n), generator=gen, device="cuda")
    tgt = torch.stack([torch.tanh(feat[:4].sum(0) * 0.5), torch.sin(feat[3:].mean(0))]).contiguous()
    u = lambda k, s: (2.0 * torch.rand(k, generator=gen, device="cuda") - 1.0) * s
    z = lambda k: torch.zeros(k, device="cuda")
    params = torch.cat([u(512, 8 ** -0.5), z(64), u(4096, 0.125), z(64), u(128, 0.125), z(2)])
    return feat, tgt, params


def _levels_data(case, seed):
    n = case["n"]
    coarse, fine = W.Layout((n // 2 + 8,) * 3, 3), W.Layout((n,) * 3, 3)
    f = Modes(coarse, seed)
    x = torch.from_numpy(coarse.coords("centre")[0]).cuda()
    rows = []
    for q in range(9):
        s = f("centre")
        rows.append(torch.where(x < 0.53, s, s + 0.7) if q < 5 else s)  # the fluid has a shock
    return coarse, fine, torch.stack(rows).contiguous()


LEVEL_PARTS = [(0, 5, "cell"), (5, 6, "xedge"), (6, 7, "yedge"), (7, 8, "zedge"), (8, 9, "vertex")]


def prepare(case, seed):
    kind = case["kind"]
    if kind == "step":
        blk = ax.Block(_step_workload(case, seed))
        start = (blk.state.clone(), blk.prim.clone())
        step = _graph(blk.step).replay if case["graph"] else blk.step
        out = torch.zeros((10,) + blk.L.shape3, dtype=F64, device="cuda") if case["tmunu"] else None
        return dict(case=case, blk=blk, start=start, step=step, tmunu=out)
    if kind == "patches":
        bt = ax.Batch(_patches(case, seed), tuning=(8, 0))
        start = (bt.state.clone(), bt.prim.clone())
        return dict(case=case, blk=bt, start=start, step=_graph(bt.step).replay if case["graph"] else bt.step,
                    tmunu=None)
    if kind == "gradient":
        w = _gradient_workload(case, seed)
        return dict(case=case, runner=adjoint.Runner(w), prim=torch.from_numpy(w.prim).cuda(),
                    gamma=torch.tensor(w.params["gamma"], dtype=F64, device="cuda"))
    if kind == "recover":
        L, params, metric, curv, A, cons, prim = _star(case, seed)
        return dict(case=case, L=L, params=params, metric=metric, curv=curv, A=A, start=(cons.clone(), prim.clone()),
                    cons=cons, prim=prim, src=torch.zeros((ax.SRC_FIELDS,) + L.shape3, dtype=F64, device="cuda"),
                    flags=torch.zeros(L.shape3, dtype=torch.uint8, device="cuda"),
                    stats=torch.zeros(6, dtype=torch.int64, device="cuda"))
    if kind == "points":
        m, prim, Bt, cons, guess = _points(case, seed)
        return dict(case=case, params=W.default_params(), metric=m, Bt=Bt.contiguous(), cons=cons, guess=guess,
                    prim=torch.empty_like(cons), flags=torch.zeros(case["n"], dtype=torch.uint8, device="cuda"))
    if kind == "levels":
        coarse, fine, cf = _levels_data(case, seed)
        return dict(case=case, coarse=coarse, fine=fine, cf=cf,
                    ff=torch.zeros((9,) + fine.shape3, dtype=F64, device="cuda"), back=torch.zeros_like(cf))
    feat, tgt, params = _train_data(case, seed)
    stdz = dict(in_shift=[0.0] * 8, in_scale=[1.0] * 8, out_shift=[0.0] * 2, out_scale=[1.0] * 2)
    return dict(case=case, feat=feat, tgt=tgt, params=params, mlp=ax.make_mlp(params, stdz), count=0,
                m=torch.zeros_like(params), v=torch.zeros_like(params),
                grad=torch.zeros(ax.MLP_NPARAMS + 1, device="cuda"),
                ws=torch.empty(ax.mlp_grad_workspace_size(case["n"]) // 4 + 1, device="cuda"))


def _gradient_workload(case, seed):
    # a smooth state: piecewise constant ones sit on limiter ties, where rounding picks the derivative's branch
    n = case["n"]
    return _curved(dict(case, nx=n, ny=n, nz=n, riemann="hlle", ct="fct", speeds="quartic", gauge="lorenz"), seed)


def run(s):
    case = s["case"]
    kind = case["kind"]
    if kind in ("step", "patches"):
        # a run of `steps` steps from the initial data
        blk = s["blk"]
        blk.state.copy_(s["start"][0])
        blk.prim.copy_(s["start"][1])
        for _ in range(case["steps"]):
            s["step"]()
        out = {"state": blk.state, "prim": blk.prim}
        if s["tmunu"] is not None:
            ax.tmunu(blk.L, blk.params, blk.metric, blk.prim, blk.state[5:8], s["tmunu"])
            out["tmunu"] = s["tmunu"]
        return out
    if kind == "gradient":
        prim = s["prim"].detach().clone().requires_grad_(True)
        gamma = s["gamma"].detach().clone().requires_grad_(True)
        loss = adjoint.density_loss_run(s["runner"], prim, gamma, case["steps"])
        loss.backward()
        return {"loss": loss.detach(), "prim": prim.grad, "gamma": gamma.grad}
    if kind == "recover":
        s["cons"].copy_(s["start"][0])
        s["prim"].copy_(s["start"][1])
        ax.c2p_src(s["L"], s["params"], s["metric"], s["curv"], s["A"], s["cons"], s["prim"], s["src"], s["flags"],
                   s["stats"])
        return {"cons": s["cons"], "prim": s["prim"], "src": s["src"], "flags": s["flags"]}
    if kind == "points":
        ax.c2p_points(s["params"], 5.0 / 3.0, s["metric"], s["Bt"], s["cons"], s["prim"], guess=s["guess"],
                      flags=s["flags"])
        return {"prim": s["prim"], "flags": s["flags"]}
    if kind == "levels":
        n, c0 = case["n"], (4, 4, 4)
        for a, b, stag in LEVEL_PARTS:
            ax.prolong(s["coarse"], s["fine"], c0, stag, s["cf"][a:b], s["ff"][a:b], (-3,) * 3, (n + 2,) * 3)
        for a, b, stag in LEVEL_PARTS:
            ax.restrict(s["coarse"], s["fine"], c0, stag, s["ff"][a:b], s["back"][a:b], c0, (n // 2 + 3,) * 3)
        return {"fine": s["ff"], "back": s["back"]}
    s["count"] += 1
    ax.mlp_grad(s["mlp"], s["feat"], s["tgt"], s["grad"], s["ws"])
    ax.mlp_adam(s["params"], s["grad"], s["m"], s["v"], 1e-3, 0.9, 0.999, 1e-8, s["count"])
    return {"grad": s["grad"], "params": s["params"], "m": s["m"], "v": s["v"]}


# Operations per zone and stage (faces, sources and recovery with separable interpolation; the hardware count of
# the framework's own kernels for PPM, scaled by the reconstruction's share for the others).
ZONE_FLOPS = {"minmod": 6500.0, "ppm": 8100.0, "mp5": 7900.0, "wenoz": 11500.0}


def work(case):
    kind = case["kind"]
    if kind in ("step", "patches"):
        # per zone and stage: the state, metric, curvature and previous primitives read, primitives and next state
        # written, and what the Runge-Kutta combination reads and writes besides (514 B for RK4, 428 B for Heun)
        if kind == "step":
            zones = case["nx"] * case["ny"] * case["nz"]
        else:
            zones = case["patches"] * sum(k ** 3 for k in SIDES) // len(SIDES)  # the mean of the sides
        rk = case.get("rk", 2)
        zs = zones * rk * case["steps"]
        more = 224.0 * zones if case.get("tmunu") else 0.0
        return {"bytes": (514.0 if rk == 4 else 428.0) * zs + more, "flops": ZONE_FLOPS[case["recon"]] * zs}
    if kind == "gradient":
        # forward (with a checkpoint of 14 fields written and read per stage) and a reverse pass of about four times
        # the forward's operations
        zs = case["n"] ** 3 * case["rk"] * case["steps"]
        return {"bytes": (428.0 * 3 + 224.0) * zs, "flops": 5.0 * ZONE_FLOPS[case["recon"]] * zs}
    if kind == "recover":
        return {"bytes": 385.0 * case["n"] ** 3, "flops": 2050.0 * case["n"] ** 3}
    if kind == "points":
        return {"bytes": (18 + 5 + (5 if case["guess"] == "warm" else 0)) * 8.0 * case["n"] + case["n"],
                "flops": 700.0 * case["n"]}
    if kind == "levels":
        n = case["n"]
        return {"bytes": 8.0 * 9 * ((n + 6) ** 3 + (n // 2 + 5) ** 3 + n ** 3 + (n // 2) ** 3),
                "flops": 9.0 * 30 * (n + 6) ** 3}
    return {"bytes": 4.0 * (10 * case["n"] + 8 * 4866), "flops": 6.0 * 4736 * case["n"]}


# ---- the equations in plain torch ---------------------------------------------------------------------------
# Fields are pairs (tensor [.., z, y, x], index of its first element per axis); a box is (lo, hi), inclusive.

SYM = ((0, 1, 2), (1, 3, 4), (2, 4, 5))


def _dot(a, b):
    return a[0] * b[0] + a[1] * b[1] + a[2] * b[2]


def _lower(g, v):
    return [g[SYM[a][0]] * v[0] + g[SYM[a][1]] * v[1] + g[SYM[a][2]] * v[2] for a in range(3)]


def _cofactors(g):
    return [g[3] * g[5] - g[4] ** 2, g[2] * g[4] - g[1] * g[5], g[1] * g[4] - g[2] * g[3], g[0] * g[5] - g[2] ** 2,
            g[1] * g[2] - g[0] * g[4], g[0] * g[3] - g[1] ** 2]


def _det(g):
    c = _cofactors(g)
    return g[0] * c[0] + g[1] * c[1] + g[2] * c[2]


def _geo(m):
    g = [m[4 + c] for c in range(6)]
    det = _det(g)
    return dict(alp=m[0], beta=[m[1], m[2], m[3]], g=g, gu=[c / det for c in _cofactors(g)], sg=torch.sqrt(det))


def _fluid(G, pr, Bt, gam):
    v = [pr[2], pr[3], pr[4]]
    vl = _lower(G["g"], v)
    B = [b / G["sg"] for b in Bt]
    Bl = _lower(G["g"], B)
    iW2, Bv, B2 = 1.0 - _dot(v, vl), _dot(B, vl), _dot(B, Bl)
    return dict(rho=pr[0], p=pr[1], v=v, vl=vl, B=B, Bl=Bl, iW2=iW2, W=1.0 / torch.sqrt(iW2), Bv=Bv, B2=B2,
                bsq=B2 * iW2 + Bv ** 2, rhoh=pr[0] + gam / (gam - 1.0) * pr[1])


def _cons(G, s):
    z, D = s["rhoh"] * s["W"] ** 2, s["rho"] * s["W"]
    S = [(z + s["B2"]) * s["vl"][j] - s["Bv"] * s["Bl"][j] for j in range(3)]
    return [G["sg"] * q for q in [D] + S + [z + s["B2"] - s["p"] - 0.5 * s["bsq"] - D]]


def _flux(G, s, D):
    U = _cons(G, s)
    vt = [G["alp"] * s["v"][a] - G["beta"][a] for a in range(3)]
    ptot, f = s["p"] + 0.5 * s["bsq"], G["alp"] * G["sg"]
    BD, iW2, Bv = s["B"][D], s["iW2"], s["Bv"]
    F = [U[0] * vt[D]]
    for j in range(3):
        F.append(U[1 + j] * vt[D] - f * (s["Bl"][j] * BD * iW2 + s["vl"][j] * Bv * BD) + (f * ptot if j == D else 0.0))
    F.append(U[4] * vt[D] + f * (ptot * s["v"][D] - Bv * BD))
    for t in ((D + 1) % 3, (D + 2) % 3):
        F.append(G["sg"] * (s["B"][t] * vt[D] - BD * vt[t]))
        U.append(G["sg"] * s["B"][t])
    return U, F


def _speeds(G, s, D, gam, kind):
    ia = 1.0 / G["alp"]
    a0, a1 = s["W"] * (s["v"][D] - G["beta"][D] * ia), -s["W"] * ia
    b0 = s["W"] * s["Bv"] * ia
    bD = (s["B"][D] + G["alp"] * b0 * a0) / s["W"]
    cs2, cA2 = gam * s["p"] / s["rhoh"], s["bsq"] / (s["rhoh"] + s["bsq"])
    w2 = cs2 + cA2 - cs2 * cA2
    g0, g1, g2 = G["gu"][SYM[D][D]] - (G["beta"][D] * ia) ** 2, -2.0 * G["beta"][D] * ia ** 2, -ia ** 2
    qa, qb, qc = (1 - w2) * a1 ** 2 - w2 * g2, 2 * (1 - w2) * a0 * a1 - w2 * g1, (1 - w2) * a0 ** 2 - w2 * g0
    sd = torch.sqrt(torch.clamp(qb ** 2 - 4 * qa * qc, min=0.0))
    q = -0.5 * (qb + torch.where(qb < 0, -sd, sd))
    r1, r2 = q / qa, qc / q
    lo, hi = torch.minimum(r1, r2), torch.maximum(r1, r2)
    if kind == "bound":
        return lo, hi
    A4, Bq = s["rhoh"] * (1 - cs2), s["rhoh"] * cs2 + s["bsq"]
    sq, tq = [a0 ** 2, 2 * a0 * a1, a1 ** 2], [bD ** 2, -2 * bD * b0, b0 ** 2]
    r = [-Bq * sq[k] + cs2 * tq[k] for k in range(3)]
    c = [A4 * sq[0] ** 2 + r[0] * g0, 2 * A4 * sq[0] * sq[1] + r[0] * g1 + r[1] * g0,
         A4 * (sq[1] ** 2 + 2 * sq[0] * sq[2]) + r[0] * g2 + r[1] * g1 + r[2] * g0,
         2 * A4 * sq[1] * sq[2] + r[1] * g2 + r[2] * g1, A4 * sq[2] ** 2 + r[2] * g2]

    def newton(x):
        step = lambda c, x: (((((c[4] * x + c[3]) * x + c[2]) * x + c[1]) * x + c[0]),
                             ((4 * c[4] * x + 3 * c[3]) * x + 2 * c[2]) * x + c[1])
        with torch.no_grad():
            x, d, done = x.detach().clone(), [k.detach() for k in c], False
            for _ in range(30):
                f, df = step(d, x)
                dx = torch.where(df != 0, f / df, 0.0)
                dx = torch.where(done, 0.0, dx) if done is not False else dx
                x = x - dx
                done = dx.abs() <= 8.9e-16 * torch.clamp(x.abs(), min=1.0)
                if bool(done.all()):
                    break
        if not c[0].requires_grad:
            return x
        f, df = step(c, x)  # zero, with the root's derivative
        return x - torch.where(df != 0, f / df.detach(), 0.0)

    return newton(lo), newton(hi)


def _mm(x, y):
    return torch.where(x * y > 0, torch.where(x.abs() <= y.abs(), x, y), 0.0 * x)


def _mc(m, c, p):
    l, r, d = c - m, p - c, 0.5 * (p - m)
    small = torch.where(l.abs() <= r.abs(), 2 * l, 2 * r)
    return torch.where(l * r > 0, torch.where(d.abs() <= small.abs(), d, small), 0.0 * l)


def _right(kind, a):
    """Value at the right face of the middle cell of a[0..4]."""
    if kind == "minmod":
        return a[2] + 0.5 * _mm(a[2] - a[1], a[3] - a[2])
    if kind == "ppm":
        s = [_mc(a[k], a[k + 1], a[k + 2]) for k in range(3)]
        fl, fr = 0.5 * (a[1] + a[2]) - (s[1] - s[0]) / 6.0, 0.5 * (a[2] + a[3]) - (s[2] - s[1]) / 6.0
        d, e = fr - fl, (fr - fl) * (a[2] - 0.5 * (fl + fr))
        r = torch.where((-d * d / 6.0 > e) & ~(e > d * d / 6.0), 3 * a[2] - 2 * fl, fr)
        return torch.where((fr - a[2]) * (a[2] - fl) <= 0, a[2], r)
    if kind == "wenoz":
        b = [13 / 12 * (a[0] - 2 * a[1] + a[2]) ** 2 + 0.25 * (a[0] - 4 * a[1] + 3 * a[2]) ** 2,
             13 / 12 * (a[1] - 2 * a[2] + a[3]) ** 2 + 0.25 * (a[1] - a[3]) ** 2,
             13 / 12 * (a[2] - 2 * a[3] + a[4]) ** 2 + 0.25 * (3 * a[2] - 4 * a[3] + a[4]) ** 2]
        w = [d * (1 + (b[0] - b[2]).abs() / (q + 1e-40)) for d, q in zip((0.1, 0.6, 0.3), b)]
        q = [2 * a[0] - 7 * a[1] + 11 * a[2], -a[1] + 5 * a[2] + 2 * a[3], 2 * a[2] + 5 * a[3] - a[4]]
        return (w[0] * q[0] + w[1] * q[1] + w[2] * q[2]) / (6 * (w[0] + w[1] + w[2]))
    m2, m1, c, p1, p2 = a
    f = (2 * m2 - 13 * m1 + 47 * c + 27 * p1 - 3 * p2) / 60
    mp = c + _mm(p1 - c, 4 * (c - m1))
    dm, d0, dp = m2 - 2 * m1 + c, m1 - 2 * c + p1, c - 2 * p1 + p2
    mm4 = lambda x, y, z, w: _mm(_mm(x, y), _mm(z, w))
    dr, dl = mm4(4 * d0 - dp, 4 * dp - d0, d0, dp), mm4(4 * d0 - dm, 4 * dm - d0, d0, dm)
    md, ul, lc = 0.5 * (c + p1) - 0.5 * dr, c + 4 * (c - m1), c + 0.5 * (c - m1) + 4 / 3 * dl
    lo = torch.maximum(torch.minimum(torch.minimum(c, p1), md), torch.minimum(torch.minimum(c, ul), lc))
    hi = torch.minimum(torch.maximum(torch.maximum(c, p1), md), torch.maximum(torch.maximum(c, ul), lc))
    return torch.where((f - c) * (f - mp) <= 0, f, f + _mm(lo - f, hi - f))


def _cut(f, box, o=(0, 0, 0)):
    t, b = f
    return t[(Ellipsis,) + tuple(slice(box[0][d] + o[d] - b[d], box[1][d] + o[d] - b[d] + 1) for d in (2, 1, 0))]


def _off(d, k):
    return tuple(k if a == d else 0 for a in range(3))


def _along(f, d, w):
    """sum_k w_k f(i - 1 + k) along axis d at every index where the stencil fits."""
    t, b = f
    dim = t.dim() - 1 - d
    n = t.shape[dim] - 3
    out = sum(w[k] * t.narrow(dim, k, n) for k in range(4))
    return out, tuple(b[a] + (1 if a == d else 0) for a in range(3))


VAL, DER = (-1 / 16, 9 / 16, 9 / 16, -1 / 16), (1 / 24, -27 / 24, 27 / 24, -1 / 24)


def _interp(f, axes, der=None):
    for d in axes:
        f = _along(f, d, DER if d == der else VAL)
    return f


class Exact:
    """Right-hand side, recovery and steps of one block from the equations."""

    def __init__(self, L, params, metric, curv, bc_cell, bc_A, A_shift, dt):
        self.L, self.p, self.dt = L, params, dt
        self.bc = (bc_cell, bc_A)
        self.shift = A_shift
        t = lambda a: (torch.as_tensor(a).cuda(), (-L.ng,) * 3)
        self.metric, self.curv = t(metric), t(curv)
        self.own = ((0, 0, 0), tuple(k - 1 for k in L.n))
        self.centre = _geo(list(_cut(_interp(self.metric, (2, 1, 0)), self.own)))

    def pad(self, t):
        return t, (-self.L.ng,) * 3

    def fill(self, t, kinds, shift=None):
        """Ghosts of the fields t [f, z, y, x], axis by axis."""
        L = self.L
        for d in range(3):
            n, dim = L.n[d], 3 - d
            own = t.narrow(dim, L.ng, n)
            at = torch.arange(-L.ng, n + L.ng + 1, device=t.device)
            if kinds[d] == "periodic":
                new = own.index_select(dim, at % n)
                if shift is not None:
                    k = torch.div(at, n, rounding_mode="floor").to(F64).reshape([-1 if a == dim else 1 for a in range(4)])
                    new = new + k * torch.as_tensor(shift[:, d], device=t.device).reshape(-1, 1, 1, 1)
            elif kinds[d] == "copy":
                new = own.index_select(dim, torch.clamp(at, 0, n - 1))
            else:
                a = torch.clamp(at, 0, n - 1)
                e0, e1 = own.index_select(dim, a), own.index_select(dim, torch.where(at <= 0, 1, n - 2))
                k = (at - a).abs().to(F64).reshape([-1 if q == dim else 1 for q in range(4)])
                new = e0 + k * (e0 - e1)
            rest = t.narrow(dim, n + 2 * L.ng + 1, t.shape[dim] - n - 2 * L.ng - 1)
            t = torch.cat([new, rest], dim)
        return t

    def fill_state(self, U):
        return torch.cat([self.fill(U[0:5], self.bc[0]), self.fill(U[5:8], self.bc[1], self.shift),
                          self.fill(U[8:9], self.bc[0])])

    def face_field(self, A, d, box):
        """Densitized field through the d faces: the curl of A."""
        a, b = (d + 1) % 3, (d + 2) % 3
        dx = self.L.dx
        D = lambda q, e: (_cut((A[0][q], A[1]), box, _off(e, 1)) - _cut((A[0][q], A[1]), box)) / dx[e]
        return D(b, a) - D(a, b)

    def centre_field(self, A, box):
        up = lambda d: (tuple(box[0][a] + (a == d) for a in range(3)), tuple(box[1][a] + (a == d) for a in range(3)))
        return [0.5 * (self.face_field(A, d, box) + self.face_field(A, d, up(d))) for d in range(3)]

    def put(self, t, value):
        """t with its owned points replaced."""
        out = t.clone()
        g, n = self.L.ng, self.L.n
        out[..., g:g + n[2], g:g + n[1], g:g + n[0]] = value
        return out

    def recover(self, U, prev, floor=False):
        """Primitives (owned points), and with floor the flags and the conserved variables after resets."""
        p, G = self.p, self.centre
        gam = p["gamma"]
        Bt = self.centre_field(self.pad(U[5:8]), self.own)
        cons = list(_cut(self.pad(U[0:5]), self.own))
        pr0 = list(_cut(self.pad(prev), self.own))
        D, S, tau = cons[0] / G["sg"], [c / G["sg"] for c in cons[1:4]], cons[4] / G["sg"]
        B = [b / G["sg"] for b in Bt]
        Su = _lower(G["gu"], S)
        S2, B2, BS = _dot(Su, S), _dot(B, _lower(G["g"], B)), _dot(B, S)
        gm = (gam - 1.0) / gam

        def residual(z, w, D, tau, S2, B2, BS):
            sw = torch.sqrt(1 - w)
            P = gm * (z * (1 - w) - D * sw)
            r1 = w * (B2 + z) ** 2 - BS ** 2 * (B2 + 2 * z) / z ** 2 - S2
            r2 = tau + D - 0.5 * B2 * (1 + w) + 0.5 * BS ** 2 / z ** 2 - z + P
            j11, j12 = 2 * (B2 + z) * (w + BS ** 2 / z ** 3), (B2 + z) ** 2
            j21, j22 = -BS ** 2 / z ** 3 - 1 + gm * (1 - w), -0.5 * B2 + gm * (-z + 0.5 * D / sw)
            return r1, r2, j11, j12, j21, j22

        with torch.no_grad():
            d = [x.detach() for x in (D, tau, S2, B2, BS)]
            v0 = [x.detach() for x in pr0]
            w = _dot(v0[2:], _lower(G["g"], v0[2:]))
            z = (v0[0] + v0[1] / gm) / (1 - w)
            done = torch.zeros_like(z, dtype=torch.bool)
            for _ in range(50):
                r1, r2, j11, j12, j21, j22 = residual(z, w, *d)
                det = j11 * j22 - j12 * j21
                dz, dw = (j12 * r2 - j22 * r1) / det, (j21 * r1 - j11 * r2) / det
                z = torch.where(done, z, z + dz)
                w = torch.where(done, w, torch.clamp(w + dw, 0.0, 1.0 - 1e-6))
                done = done | (torch.maximum(dz.abs() / z, dw.abs()) < 1e-14)
                if bool(done.all()):
                    break
        if U.requires_grad:
            r1, r2, j11, j12, j21, j22 = residual(z, w, D, tau, S2, B2, BS)
            j = [x.detach() for x in (j11, j12, j21, j22)]
            det = j[0] * j[3] - j[1] * j[2]
            z, w = z + (j[1] * r2 - j[3] * r1) / det, w + (j[2] * r1 - j[0] * r2) / det
        W_ = 1 / torch.sqrt(1 - w)
        rho = D / W_
        P = gm * (z * (1 - w) - rho)
        v = [(Su[a] + BS * B[a] / z) / (z + B2) for a in range(3)]
        out = torch.stack([rho, P] + v)
        if not floor:
            return out, Bt
        low = cons[0] < G["sg"] * p["rho_atm"]
        none = ~low & (B2 <= 0) & (S2 > tau * (tau + 2 * D))
        reset = low | none
        atm = torch.zeros_like(out)
        atm[0], atm[1] = p["rho_atm"], p["k_atm"] * p["rho_atm"] ** gam
        out = torch.where(reset, atm, out)
        new = torch.where(reset, torch.stack(_cons(G, _fluid(G, atm, Bt, gam))), torch.stack(cons))
        flags = torch.where(low, 4, torch.where(none, 13, 0)).to(torch.uint8)
        return out, Bt, new, flags

    def sources(self, prim, Bt):
        """Densitized sources of S_j and tau at the owned cells."""
        G = self.centre
        s = _fluid(G, prim, Bt, self.p["gamma"])
        T00, T0, T = _stress(G, s)
        K = list(_cut(_interp(self.curv, (2, 1, 0)), self.own))
        dm = [list(_cut(_interp(self.metric, (2, 1, 0), d), self.own) / self.L.dx[d]) for d in range(3)]
        be, bl, f = G["beta"], _lower(G["g"], G["beta"]), G["alp"] * G["sg"]
        out = []
        for d in range(3):
            dal, db, dg = dm[d][0], dm[d][1:4], dm[d][4:]
            x = _lower(dg, be)
            d00 = -2 * G["alp"] * dal + _dot(be, x) + 2 * _dot(bl, db)
            y = _lower(G["g"], db)
            tot = 0.5 * T00 * d00 + sum(T0[a] * (x[a] + y[a]) for a in range(3))
            tot = tot + 0.5 * sum(T[SYM[a][b]] * dg[SYM[a][b]] for a in range(3) for b in range(3))
            out.append(f * tot)
        e = sum((T00 * be[a] * be[b] + 2 * T0[a] * be[b] + T[SYM[a][b]]) * K[SYM[a][b]] for a in range(3) for b in range(3))
        e = e - sum((T00 * be[a] + T0[a]) * dm[a][0] for a in range(3))
        return out + [f * e]

    def faces(self, D, prim, A, bc):
        p, L = self.p, self.L
        wide = 3 if p["ct"] == "uct" else 1
        t1, t2 = (D + 1) % 3, (D + 2) % 3
        lo = tuple(0 if a == D else -wide for a in range(3))
        hi = tuple(L.n[a] if a == D else L.n[a] + wide - 2 for a in range(3))
        box = (lo, hi)
        G = _geo(list(_cut(_interp(self.metric, (t2, t1)), box)))
        Bn = self.face_field(A, D, box)
        var = [(prim[0][q], prim[1]) for q in range(5)] + [(bc[0][t], bc[1]) for t in (t1, t2)]
        side = []
        for s in (0, 1):
            X = []
            for f in var:
                a = [_cut(f, box, _off(D, (k - 3) if s == 0 else (2 - k))) for k in range(5)]
                X.append(_right(p["recon"], a))
            cell = [_cut(f, box, _off(D, s - 1)) for f in var]
            v2 = _dot(X[2:5], _lower(G["g"], X[2:5]))
            bad = ~((X[0] > 0) & (X[1] > 0) & (v2 < 1))
            X = [torch.where(bad, c, x) for c, x in zip(cell, X)]
            Bt = [None] * 3
            Bt[D], Bt[t1], Bt[t2] = Bn, X[5], X[6]
            st = _fluid(G, X, Bt, p["gamma"])
            side.append(_flux(G, st, D) + _speeds(G, st, D, p["gamma"], p["speeds"]) + (X,))
        (UL, FL, mL, pL, XL), (UR, FR, mR, pR, XR) = side
        zero = torch.zeros_like(mL)
        cp = torch.maximum(zero, torch.maximum(pL, pR))
        cm = -torch.minimum(zero, torch.minimum(mL, mR))
        if p["riemann"] == "lxf":
            c = torch.maximum(cp, cm)
            F = [0.5 * (fl + fr - c * (ur - ul)) for fl, fr, ul, ur in zip(FL, FR, UL, UR)]
        else:
            F = [(cm * fr + cp * fl - cp * cm * (ur - ul)) / (cp + cm) for fl, fr, ul, ur in zip(FL, FR, UL, UR)]
        vb = {}
        for t in (t1, t2):
            vl, vr = (G["alp"] * X[2 + t] - G["beta"][t] for X in (XL, XR))
            vb[t] = ((cp * vl + cm * vr) / (cp + cm), lo)
        return dict(F=[(f, lo) for f in F], cp=(cp, lo), cm=(cm, lo), Bn=(Bn, lo), vb=vb)

    def edge_field(self, fc, c):
        a, b = (c + 1) % 3, (c + 2) % 3
        box = self.own
        if self.p["ct"] == "fct":
            slot = lambda D, t: fc[D]["F"][5 if t == (D + 1) % 3 else 6]
            q = lambda f, e: _cut(f, box) + _cut(f, box, _off(e, -1))
            return 0.25 * (-q(slot(a, b), b) + q(slot(b, a), a))

        def term(d, fd):
            # the problem along d at the edge, from the fd faces in the row through it
            lr = []
            for f in (fc[fd]["vb"][d], fc[fd]["Bn"]):
                a6 = [_cut(f, box, _off(d, k - 3)) for k in range(6)]
                lr.append((_right("ppm", a6[0:5]), _right("ppm", a6[5:0:-1])))
            (vl, vr), (bl, br) = lr
            cp, cm = (torch.maximum(_cut(fc[d][k], box), _cut(fc[d][k], box, _off(fd, -1))) for k in ("cp", "cm"))
            return (cp * vl * bl + cm * vr * br - cp * cm * (br - bl)) / (cp + cm)

        return -term(a, b) + term(b, a)

    def rhs(self, U, prim, Bt):
        """Right-hand side of the nine fields at the owned points; U and prim have their ghosts."""
        L, p, own = self.L, self.p, self.own
        A, psi = self.pad(U[5:8]), self.pad(U[8])
        wide = ((-L.ng,) * 3, tuple(k + L.ng - 1 for k in L.n))
        bc = (torch.stack(self.centre_field(A, wide)), (-L.ng,) * 3)
        fc = [self.faces(D, self.pad(prim), A, bc) for D in range(3)]
        src = [0.0] + self.sources(list(_cut(self.pad(prim), own)), Bt)
        out = []
        for c in range(5):
            div = sum((_cut(fc[d]["F"][c], own, _off(d, 1)) - _cut(fc[d]["F"][c], own)) / L.dx[d] for d in range(3))
            out.append(src[c] - div)
        E = [self.edge_field(fc, c) for c in range(3)]
        if p["gauge"] == "algebraic":
            return torch.stack(out + [-e for e in E] + [torch.zeros_like(E[0])])
        vb = ((-1,) * 3, tuple(L.n))
        G = _geo(list(_cut(self.metric, vb)))
        Av = [0.5 * (_cut((A[0][d], A[1]), vb) + _cut((A[0][d], A[1]), vb, _off(d, -1))) for d in range(3)]
        ps = _cut(psi, vb)
        GA = (G["alp"] * ps / G["sg"] - _dot(G["beta"], Av), vb[0])
        up = _lower(G["gu"], Av)
        FP = [(G["alp"] * G["sg"] * up[d] - G["beta"][d] * ps, vb[0]) for d in range(3)]
        out += [-E[d] - (_cut(GA, own, _off(d, 1)) - _cut(GA, own)) / L.dx[d] for d in range(3)]
        div = sum((_cut(FP[d], own, _off(d, 1)) - _cut(FP[d], own, _off(d, -1))) / (2 * L.dx[d]) for d in range(3))
        out.append(-div - p["xi"] / self.dt * _cut((self.metric[0][0], self.metric[1]), own) * _cut(psi, own))
        return torch.stack(out)

    def stage(self, U, prim):
        """(right-hand side at the owned points, primitives with ghosts)."""
        new, Bt = self.recover(U, prim)
        prim = self.fill(self.put(prim, new), self.bc[0])
        return self.rhs(U, prim, Bt), prim

    def step(self, U, prim, rk):
        own = lambda t: _cut(self.pad(t), self.own)
        nxt = lambda v: self.fill_state(self.put(U, v))
        dt, U0 = self.dt, own(U)
        k1, prim = self.stage(U, prim)
        if rk == 2:
            U1 = nxt(U0 + dt * k1)
            k2, prim = self.stage(U1, prim)
            return nxt(0.5 * U0 + 0.5 * own(U1) + 0.5 * dt * k2), prim
        k2, prim = self.stage(nxt(U0 + 0.5 * dt * k1), prim)
        k3, prim = self.stage(nxt(U0 + 0.5 * dt * k2), prim)
        k4, prim = self.stage(nxt(U0 + dt * k3), prim)
        return nxt(U0 + dt / 6 * (k1 + 2 * k2 + 2 * k3 + k4)), prim

    def initial(self, A, psi, prim):
        A = torch.as_tensor(A).cuda()
        Bt = self.centre_field(self.pad(A), self.own)
        pr = list(_cut(self.pad(prim), self.own))
        cons = torch.stack(_cons(self.centre, _fluid(self.centre, pr, Bt, self.p["gamma"])))
        U = torch.zeros((5,) + self.L.shape3, dtype=F64, device="cuda")
        return torch.cat([self.fill(self.put(U, cons), self.bc[0]), A, torch.as_tensor(psi).cuda()])

    def tmunu(self, U, prim):
        L = self.L
        box = ((0,) * 3, tuple(L.n))
        wide = ((-1,) * 3, tuple(L.n))
        f = torch.cat([_cut(self.pad(prim), wide), torch.stack(self.centre_field(self.pad(U[5:8]), wide))])
        for dim in (1, 2, 3):
            k = f.shape[dim] - 1
            f = 0.5 * (f.narrow(dim, 0, k) + f.narrow(dim, 1, k))
        m = list(_cut(self.metric, box))
        G = _geo(m)
        T00, T0, T = _stress(G, _fluid(G, list(f[0:5]), list(f[5:8]), self.p["gamma"]))
        bl = _lower(G["g"], G["beta"])
        g4 = [[-G["alp"] ** 2 + _dot(bl, G["beta"])] + bl] + [[bl[a]] + [G["g"][SYM[a][b]] for b in range(3)] for a in range(3)]
        Tu = [[T00] + T0] + [[T0[a]] + [T[SYM[a][b]] for b in range(3)] for a in range(3)]
        X = [[sum(Tu[a][c] * g4[c][b] for c in range(4)) for b in range(4)] for a in range(4)]
        rows = [sum(g4[a][c] * X[c][b] for c in range(4)) for a in range(4) for b in range(a, 4)]
        out = torch.zeros((10,) + L.shape3, dtype=F64, device="cuda")
        g = L.ng
        out[:, g:g + L.n[2] + 1, g:g + L.n[1] + 1, g:g + L.n[0] + 1] = torch.stack(rows)
        return out


def _stress(G, s):
    """T^00, T^0i, T^ij (six components)."""
    al, be = G["alp"], G["beta"]
    u0, b0 = s["W"] / al, s["W"] * s["Bv"] / al
    u = [s["W"] * (s["v"][a] - be[a] / al) for a in range(3)]
    b = [(s["B"][a] + al * b0 * u[a]) / s["W"] for a in range(3)]
    e, pt = s["rhoh"] + s["bsq"], s["p"] + 0.5 * s["bsq"]
    T0 = [e * u0 * u[a] + pt * be[a] / al ** 2 - b0 * b[a] for a in range(3)]
    T = [e * u[a] * u[c] + pt * (G["gu"][SYM[a][c]] - be[a] * be[c] / al ** 2) - b[a] * b[c] for a in range(3)
         for c in range(a, 3)]
    return e * u0 ** 2 - pt / al ** 2 - b0 ** 2, T0, T


def _exact_of(w):
    return Exact(w.layout, w.params, w.metric, w.curv, w.bc_cell, w.bc_A, w.A_shift, w.dt)


def _exact_steps(w, steps):
    E = _exact_of(w)
    prim = torch.from_numpy(w.prim).cuda()
    U = E.initial(w.A, w.psi, prim)
    for _ in range(steps):
        U, prim = E.step(U, prim, w.rk)
    return E, U, prim


def _exact_levels(case, seed):
    coarse, fine, cf = _levels_data(case, seed)
    n, c0 = case["n"], 4
    f = torch.arange(-4, n + 4, device="cuda")  # whole parents; the box is cut from it
    par = c0 + torch.div(f, 2, rounding_mode="floor") + coarse.ng
    ff = torch.zeros((9,) + fine.shape3, dtype=F64, device="cuda")

    def weights(vertex):
        """Row f: the weights of the coarse points parent - 1 .. parent + 2."""
        odd = (f % 2 == 1)[:, None]
        e = lambda *v: torch.tensor(v, dtype=F64, device="cuda")
        if vertex:
            return torch.where(odd, e(-1, 9, 9, -1) / 16, e(0, 1, 0, 0))
        return torch.where(odd, e(-1, 8, 1, 0) / 8, e(1, 8, -1, 0) / 8)

    for a, b, stag in LEVEL_PARTS:
        out = cf[a:b]
        for d in range(3):
            w, dim = weights(ax.STAG[stag][d]), 3 - d
            shape = [-1 if q == dim else 1 for q in range(4)]
            out = sum(w[:, k].reshape(shape) * out.index_select(dim, par - 1 + k) for k in range(4))
        if stag == "cell":
            u = cf[a:b]
            mx = torch.nn.functional.max_pool3d(u, 3, 1, 1)
            mn = -torch.nn.functional.max_pool3d(-u, 3, 1, 1)
            sl = [_mm(torch.roll(u, -1, 3 - d) - u, u - torch.roll(u, 1, 3 - d)) for d in range(3)]
            up = lambda t: t.index_select(1, par).index_select(2, par).index_select(3, par)
            sign = lambda d: torch.where(f % 2 == 1, 0.25, -0.25).to(F64).reshape([-1 if q == 3 - d else 1 for q in range(4)])
            bad = ((out > up(mx)) | (out < up(mn))).double()
            bad = torch.nn.functional.max_pool3d(bad, 2, 2)  # one decision per parent
            bad = bad.repeat_interleave(2, 1).repeat_interleave(2, 2).repeat_interleave(2, 3)
            lin = up(u) + sum(sign(d) * up(sl[d]) for d in range(3))
            out = torch.where(bad > 0, lin, out)
        ff[a:b, :n + 6, :n + 6, :n + 6] = out[:, 1:-1, 1:-1, 1:-1]
    back = torch.zeros_like(cf)
    g, h = fine.ng, n // 2
    for a, b, stag in LEVEL_PARTS:
        t = ff[a:b, g:g + n, g:g + n, g:g + n]
        for d in range(3):
            dim = 3 - d
            even = t.index_select(dim, torch.arange(0, n, 2, device="cuda"))
            t = even if ax.STAG[stag][d] else 0.5 * (even + t.index_select(dim, torch.arange(1, n, 2, device="cuda")))
        o = c0 + coarse.ng
        back[a:b, o:o + h, o:o + h, o:o + h] = t
    return {"fine": ff, "back": back}


def _exact_train(case, seed):
    feat, tgt, params = _train_data(case, seed)
    p = params.double().requires_grad_(True)
    w1, b1, w2, b2, w3, b3 = torch.split(p, [512, 64, 4096, 64, 128, 2])
    h = torch.relu(w1.reshape(64, 8) @ feat.double() + b1[:, None])
    h = torch.relu(w2.reshape(64, 64) @ h + b2[:, None])
    y = w3.reshape(2, 64) @ h + b3[:, None]
    loss = 0.5 * ((y - tgt.double()) ** 2).sum() / case["n"]
    (g,) = torch.autograd.grad(loss, p)
    new = p.detach() - 1e-3 * g / (g.abs() + 1e-8)
    return {"grad": torch.cat([g, loss.detach().reshape(1)]), "params": new, "m": 0.1 * g, "v": 0.001 * g ** 2}


def exact(case, seed):
    kind = case["kind"]
    if kind == "step":
        E, U, prim = _exact_steps(_step_workload(case, seed), case["steps"])
        out = {"state": U, "prim": prim}
        if case["tmunu"]:
            out["tmunu"] = E.tmunu(U, prim)
        return out
    if kind == "patches":
        done = [_exact_steps(w, case["steps"])[1:] for w in _patches(case, seed)]
        return {k: torch.cat([d[i].flatten(1) for d in done], 1) for i, k in enumerate(("state", "prim"))}
    if kind == "gradient":
        w = _gradient_workload(case, seed)
        prim = torch.from_numpy(w.prim).cuda().requires_grad_(True)
        gamma = torch.tensor(w.params["gamma"], dtype=F64, device="cuda", requires_grad=True)
        w.params = dict(w.params, gamma=gamma)
        E = _exact_of(w)
        U, pr = E.initial(w.A, w.psi, prim), prim
        for _ in range(case["steps"]):
            U, pr = E.step(U, pr.detach(), w.rk)
        rho = E.recover(U, pr.detach())[0][0]
        loss = torch.sqrt((rho ** 2).sum() * (w.layout.dx[0] * w.layout.dx[1] * w.layout.dx[2]))
        loss.backward()
        return {"loss": loss.detach(), "prim": prim.grad, "gamma": gamma.grad}
    if kind == "recover":
        L, params, metric, curv, A, cons, prim = _star(case, seed)
        E = Exact(L, params, metric, curv, ("copy",) * 3, ("copy",) * 3, None, 1.0)
        U = torch.cat([cons, A, torch.zeros_like(A[:1])])
        out, Bt, new, flags = E.recover(U, prim, floor=True)
        src = torch.zeros((ax.SRC_FIELDS,) + L.shape3, dtype=F64, device="cuda")
        src[0:4] = E.put(src[0:4], torch.stack(E.sources(list(out), Bt)))
        box = ((0, 0, 0), (L.n[0], L.n[1] - 1, L.n[2] - 1))
        g = L.ng
        src[4:14, g:g + L.n[2], g:g + L.n[1], g:g + L.n[0] + 1] = _cut(_interp(E.metric, (2, 1)), box)
        keep = torch.zeros(L.shape3, dtype=torch.uint8, device="cuda")
        return {"cons": E.put(cons, new), "prim": E.put(prim, out), "src": src, "flags": E.put(keep, flags)}
    if kind == "points":
        return {"prim": _points(case, seed)[1], "flags": torch.zeros(case["n"], dtype=torch.uint8, device="cuda")}
    if kind == "levels":
        return _exact_levels(case, seed)
    return _exact_train(case, seed)
