"""The workloads whose speed is measured, from the smallest call to the largest.

Sizes are this repository's own: the meshes, flows, limiters, CFL numbers and
batch sizes of the benchmark, the tests and the evaluation runs, and drawn
variants of them (odd root grids, other depths, other combinations of options).

A case is a dict of plain values.  Its "kind":

  steps     a solver with a mesh and a state; a pass is `steps` SSP-RK3 steps as
            a time loop takes them, then the state brought back on the device
  adapt     one turn of a run with adaptive refinement: the indicator, flags (a
            refined region on a given path, so that every seed has the same
            meshes), refinement and transfer, then `steps` steps with statistics
  sensors   the per-element sensors that drive refinement: the features, the
            modal indicator and the learned one
  train     loss and gradient of the learned indicator's network on a batch
  network   the network on stored features
"""
import functools
import math

import numpy as np
import torch

import paper_2607_06045_amd as P

LIMITERS = {"none": P.LIMIT_NONE, "positivity": P.LIMIT_POSITIVITY, "local": P.LIMIT_LOCAL,
            "combined": P.LIMIT_COMBINED, "lowsol": P.LIMIT_LOCAL_LOWORDER}
GAMMA = {"jet": 5.0 / 3.0}
BOX = {"vortex": (0.0, 0.0, 1.0, 1.0), "blast": (-1.0, -1.0, 2.0, 2.0), "shear": (-1.0, -1.0, 2.0, 2.0),
       "quadrants": (0.0, 0.0, 1.0, 1.0), "jet": (-0.5, -0.5, 1.0, 1.0), "dmr": (0.0, 0.0, 3.25, 1.0)}


def case_of(name, kind, flow="blast", N=3, nx=64, ny=64, levels=0, width=0.3, limiter="positivity",
            precision="fp64", cfl=0.5, steps=5, loop="plain", batch=0):
    c = {"kind": kind, "batch": batch} if kind in ("train", "network") else \
        {"kind": kind, "flow": flow, "N": N, "nx": nx, "ny": ny, "levels": levels, "width": width}
    if kind in ("steps", "adapt"):
        c.update(limiter=limiter, precision=precision, cfl=cfl, steps=steps)
    if kind == "steps":
        c["loop"] = loop
    return dict(c, name=name) if name else c


def listed():
    return [
        # the smallest mesh of the tests (304 leaves): launches and latency
        case_of("step_vortex304", "steps", "vortex", 3, 16, 16, 1, 0.125),
        # the benchmark's middle workload, in one launch per stage
        case_of("step_blast22k", "steps", "blast", 3, 64, 64, 3, 0.3),
        # the benchmark's shear layer in the mixed precision mode
        case_of("step_shear59k_mixed", "steps", "shear", 3, 128, 128, 3, 0.0175, precision="mixed"),
        # the benchmark's headline: 6.2 million nodes, more than the last-level cache holds
        case_of("step_quadrants247k", "steps", "quadrants", 4, 256, 256, 2, 0.022),
        # an odd root grid at N = 4 with many mortars
        case_of("step_blast_n4_odd", "steps", "blast", 4, 45, 37, 3, 0.4),
        # the other limiters as the benchmark runs them on the blast
        case_of("step_blast22k_local", "steps", "blast", 3, 64, 64, 3, 0.3, "local"),
        case_of("step_blast22k_lowsol", "steps", "blast", 3, 64, 64, 3, 0.3, "lowsol", cfl=0.4),
        # the jet: inflow boundaries, the other volume flux, blended limiting, dt by the host
        case_of("step_jet_combined", "steps", "jet", 3, 128, 128, 2, 0.06, "combined", cfl=0.9, steps=3, loop="host_dt"),
        # the double Mach reflection: walls and inflow, N = 4, local limiting, dt by the host
        case_of("step_dmr_local", "steps", "dmr", 4, 256, 80, 0, 0.0, "local", cfl=0.9, steps=3, loop="host_dt"),
        # a blast with its mesh adapted every five steps
        case_of("adapt_blast22k", "adapt", "blast", 3, 64, 64, 3, 0.3),
        # the sensors on the headline mesh
        case_of("sensors_quadrants247k", "sensors", "quadrants", 4, 256, 256, 2, 0.022),
        # one batch of the network's training as the evaluation runs train it
        case_of("train_8192", "train", batch=8192),
    ]


def draw(rng):
    def log_int(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    r = rng.random()
    if r < 0.12:
        return case_of(None, "train", batch=log_int(100, 60000))
    if r < 0.2:
        return case_of(None, "network", batch=log_int(1000, 300000))
    kind = "sensors" if r < 0.32 else "adapt" if r < 0.42 else "steps"
    flow = rng.choice(["vortex", "blast", "shear", "quadrants"] + (["jet", "dmr"] if kind == "steps" else []))
    N = rng.choice([3, 4])
    limiter = rng.choice(["none", "positivity", "positivity", "positivity", "local", "combined", "lowsol"])
    if flow in ("jet", "dmr"):
        limiter = "combined" if flow == "jet" else "local"
    elif kind == "adapt":
        limiter = "positivity"
    elif limiter == "none" and flow != "vortex":
        limiter = "positivity"
    levels = rng.choice([0, 1, 2, 3])
    width = {"vortex": 0.125, "blast": 0.3, "shear": 0.0175, "quadrants": 0.022, "jet": 0.06, "dmr": 0.0}[flow]
    # the root grid: from a few elements a side up to a few million nodes, fewer
    # where a node costs several times the plain method's
    most = [300, 256, 180, 100][levels] if limiter == "positivity" and kind != "adapt" else [110, 110, 55, 36][levels]
    nx = log_int(12, most)
    ny = max(8, int(nx * rng.uniform(0.6, 1.0)))
    if flow == "dmr":
        levels, ny = 0, max(5, int(round(nx / 3.25)))
    precision = rng.choice(["fp64", "fp64", "mixed"])
    cfl = 0.4 if limiter == "lowsol" else 0.9 if flow in ("jet", "dmr") else 0.5
    loop = "host_dt" if flow in ("jet", "dmr") or limiter == "lowsol" and rng.random() < 0.5 else \
        rng.choice(["plain", "plain", "stats"])
    return case_of(None, kind, flow, N, nx, ny, levels, width, limiter, precision, cfl, rng.choice([2, 3, 5]), loop)


# --------------------------------------------------------------------------
# meshes
# --------------------------------------------------------------------------
def wants(flow, width, x, y, hx, hy):
    """Which leaves (centre x, y, size hx, hy) the flow's start refines."""
    if flow == "blast":
        return x * x + y * y <= width * width
    if flow == "vortex":
        return (abs(x - 0.5) < width) & (abs(y - 0.5) < width)
    if flow == "shear":
        return abs(abs(y) - 0.5) < width + 0.5 * hy
    if flow == "quadrants":
        def near(t, h):
            return np.minimum(np.minimum(abs(t), abs(t - 0.5)), abs(t - 1.0)) < width + 0.5 * h
        return near(x, hx) | near(y, hy)
    return (x < -0.3) & (abs(y) < width + hy)  # jet: the inflow region


@functools.lru_cache(maxsize=32)
def leaves(flow, nx, ny, levels, width):
    """Leaf list (level, ix, iy): the nx x ny root grid, refined `levels` times."""
    x0, y0, Lx, Ly = BOX[flow]
    iy, ix = (a.ravel().astype(np.int32) for a in np.meshgrid(np.arange(ny), np.arange(nx), indexing="ij"))
    level = np.zeros(nx * ny, np.int8)
    for k in range(levels):
        hx, hy = Lx / (nx << level.astype(np.int64)), Ly / (ny << level.astype(np.int64))
        ask = (level == k) & wants(flow, width, x0 + (ix + 0.5) * hx, y0 + (iy + 0.5) * hy, hx, hy)
        level, ix, iy, _, _ = P.adapt_leaves(level, ix, iy, nx, ny, ask.astype(np.int8))
    return level, ix, iy


def mesh_of(c):
    return leaves(c["flow"], c["nx"], c["ny"], c["levels"], c["width"])


# --------------------------------------------------------------------------
# states (conservative variables; seeded)
# --------------------------------------------------------------------------
def conservative(rho, v1, v2, p, g):
    return torch.stack([rho, rho * v1, rho * v2, p / (g - 1.0) + 0.5 * rho * (v1 * v1 + v2 * v2)], dim=1).contiguous()


DMR_POST = (8.0, 8.25 * math.cos(math.pi / 6), -8.25 * math.sin(math.pi / 6), 116.5)
DMR_PRE = (1.4, 0.0, 0.0, 1.0)


def initial(flow, x, y, seed):
    """The flow's start at the nodes x, y ([E, n, n]), [E, 4, n, n]."""
    r = np.random.RandomState(seed % (1 << 31)).uniform(size=24)
    one = torch.ones_like(x)
    if flow == "blast":  # a Gaussian of pressure, centre and strength by the seed
        s2 = 2 * 0.06 ** 2
        xc, yc, e = 0.02 * (r[0] - 0.5), 0.02 * (r[1] - 0.5), 0.8 + 0.4 * r[2]
        return conservative(one, 0 * one, 0 * one,
                            1e-5 + 0.4 * e * torch.exp(-((x - xc) ** 2 + (y - yc) ** 2) / s2) / (math.pi * s2), 1.4)
    if flow == "vortex":  # isentropic vortex with a perturbed density
        xb, yb = (x - 0.5 - 0.02 * (r[0] - 0.5)) / 0.1, (y - 0.5 - 0.02 * (r[1] - 0.5)) / 0.1
        r2 = xb * xb + yb * yb
        rho = (1.0 - 10.0 * torch.exp(1.0 - r2) / (11.2 * math.pi ** 2)) ** 2.5
        s = 5.0 / (2 * math.pi) * torch.exp(0.5 * (1.0 - r2))
        p = rho ** 1.4
        g = torch.Generator(device=x.device).manual_seed(seed)
        rho = rho + 1e-3 * (2 * torch.rand(x.shape, dtype=x.dtype, device=x.device, generator=g) - 1)
        return conservative(rho, -s * yb, s * xb, p, 1.4)
    if flow == "shear":  # two layers and a transverse wave
        inside = abs(y) < 0.5
        return conservative(torch.where(inside, 1.0, 0.5).to(x.dtype), torch.where(inside, 0.5, -0.5).to(x.dtype),
                            (0.05 + 0.1 * r[0]) * torch.sin(2 * math.pi * (x + r[1])), 2.5 * one, 1.4)
    if flow == "quadrants":  # four constant states, meeting in four Riemann problems a side
        q = (x >= 0.5).long() + 2 * (y >= 0.5).long()
        pick = lambda lo, hi, k: torch.tensor(lo + (hi - lo) * r[k:k + 4], dtype=x.dtype, device=x.device)[q]  # noqa: E731
        return conservative(pick(0.1, 1.5, 0), pick(-1.0, 1.0, 8), pick(-1.0, 1.0, 12), pick(0.03, 1.5, 4), 1.4)
    if flow == "jet":  # the ambient gas, at rest up to a small random pressure
        return conservative(0.5 * one, 0 * one, 0 * one, 0.4127 * (1 + 1e-3 * torch.sin(2 * math.pi * (x + y + r[0]))),
                            GAMMA["jet"])
    left = x < 1.0 / 6.0 + 0.05 * r[0] + y / math.sqrt(3.0)  # dmr: the oblique incident shock
    return torch.where(left[:, None], conservative(*(v * one for v in DMR_POST), 1.4),
                       conservative(*(v * one for v in DMR_PRE), 1.4))


def point(rho, v1, v2, p, g):
    return np.array([rho, rho * v1, rho * v2, p / (g - 1.0) + 0.5 * rho * (v1 * v1 + v2 * v2)])


def solver_of(c, seed):
    flow, g = c["flow"], GAMMA.get(c["flow"], 1.4)
    kw = {}
    if flow == "jet":
        CH = P.BC_CHARACTERISTIC
        amb = point(0.5, 0.0, 0.0, 0.4127, g)
        kw = dict(bc=[CH, CH, P.BC_PERIODIC, P.BC_PERIODIC], ext=np.stack([amb] * 4), volume_flux=P.FLUX_CHANDRASHEKAR)
    elif flow == "dmr":
        post, pre = point(*DMR_POST, g), point(*DMR_PRE, g)
        kw = dict(bc=[P.BC_CHARACTERISTIC] * 4, ext=np.stack([post, pre, post, pre]))
    limiter = c.get("limiter", "positivity")
    s = P.Solver(c["N"], gamma=g, precision=P.MIXED if c.get("precision") == "mixed" else P.FP64,
                 limiter=LIMITERS[limiter], dt_mode=P.DT_LOWORDER if limiter == "lowsol" else P.DT_IDP, **kw)
    x0, y0, Lx, Ly = BOX[flow]
    s.set_mesh(*mesh_of(c), x0, y0, Lx, Ly, c["nx"], c["ny"])
    x, y = s.node_coords()
    if kw:  # boundary states node by node: the jet's inflow, the wall of the double Mach reflection
        e, f, k = s.boundary_nodes().T
        b, a = np.where(f < 2, k, np.where(f == 2, 0, c["N"])), np.where(f >= 2, k, np.where(f == 0, 0, c["N"]))
        bx, by = x[e, b, a], y[e, b, a]
        kind = np.full(len(e), P.BC_CHARACTERISTIC, np.int8)
        if flow == "jet":
            ext = np.tile(amb, (len(e), 1))
            ext[(f == 0) & (abs(by) <= 0.05)] = point(5.0, 800.0, 0.0, 0.4127, g)
        else:
            kind[(f == 2) & (bx >= 1.0 / 6.0)] = P.BC_WALL
            ext = np.where((bx < 1.0 / 6.0 + by / np.sqrt(3.0))[:, None], post, pre)
            ext[f == 2] = post
        s.set_boundary_states(kind, ext)
    s.upload(initial(flow, torch.from_numpy(x).cuda(), torch.from_numpy(y).cuda(), seed))
    return s


def weights_of(seed):
    """He-uniform weights of the 16-64-64-1 network in the library's order."""
    r = np.random.RandomState(seed % (1 << 31))
    w = [r.uniform(-1, 1, k) * np.sqrt(6.0 / fan) for k, fan in ((1024, 16), (4096, 64), (64, 64))]
    small = [0.1 * r.uniform(-1, 1, k) for k in (64, 64, 1)]
    return np.concatenate([w[0], small[0], w[1], small[1], w[2], small[2]]).astype(np.float32)


def batch_of(c, seed):
    """Features (four groups of four energy fractions, falling off by decades)
    and targets in [0, 0.5]."""
    g = torch.Generator(device="cuda").manual_seed(seed)
    e = torch.exp(-6.0 * torch.rand((c["batch"], 4, 4), device="cuda", generator=g) * torch.arange(4, device="cuda"))
    return (e / e.sum(2, keepdim=True)).reshape(-1, 16).contiguous(), \
        0.5 * torch.rand(c["batch"], device="cuda", generator=g)


def prepare(case, seed):
    if case["kind"] in ("train", "network"):
        s = P.Solver(3)
        s.mlp_set_weights(weights_of(seed))
        x, t = batch_of(case, seed)
        return {"case": case, "solver": s, "x": x, "t": t}
    s = solver_of(case, seed)
    if case["kind"] == "sensors":
        for _ in range(3):  # a flow on its way, not its start
            s.step(0.5, stats=False)
        s.mlp_set_weights(weights_of(seed))
    return {"case": case, "solver": s, "turn": 0}


def told(st):
    return {"dt": st["dt"], "violations": st["violations"], "fv_inadmissible": st["fv_inadmissible"]}


def run(state):
    c, s = state["case"], state["solver"]
    if c["kind"] == "train":
        grad, loss = s.mlp_grad(state["x"], state["t"])
        return {"grad": grad, "loss": loss}
    if c["kind"] == "network":
        return {"y": s.mlp_forward(state["x"])}
    if c["kind"] == "sensors":
        return {"features": s.features(device=True), "modal": s.indicator(P.IND_HENNEMANN, device=True),
                "learned": s.indicator(P.IND_MLP, device=True)}
    out = {}
    if c["kind"] == "adapt":
        level, ix, iy = s.mesh()
        out["modal"] = s.indicator(P.IND_HENNEMANN)
        x0, y0, Lx, Ly = BOX[c["flow"]]
        state["turn"] += 1
        dx, dy = 0.02 * Lx * math.cos(state["turn"]), 0.02 * Ly * math.sin(state["turn"])
        hx, hy = Lx / (c["nx"] << level.astype(np.int64)), Ly / (c["ny"] << level.astype(np.int64))
        here = wants(c["flow"], c["width"], x0 + (ix + 0.5) * hx - dx, y0 + (iy + 0.5) * hy - dy, hx, hy)
        st = s.refine_coarsen(P.amr_flags(here, level, 0, 0, 0.5, c["levels"], 0.5))
        out.update(n_refined=st["n_refined"], n_coarsened=st["n_coarsened"], level=s.mesh()[0])
    said = []
    for _ in range(c["steps"]):
        if c["kind"] == "adapt" or c["loop"] == "stats":
            said.append(told(s.step(c["cfl"])))
        elif c["loop"] == "host_dt":
            said.append(told(s.step_dt(s.max_dt(c["cfl"]))))
        else:
            s.step(c["cfl"], stats=False)
    return dict(out, stats=said, u=s.download(device=True))


def work(case):
    if case["kind"] in ("train", "network"):
        # products of the three layers; the gradient takes them three times
        B, products = case["batch"], 2 * (16 * 64 + 64 * 64 + 64)
        if case["kind"] == "train":
            return {"bytes": 4 * (17 * B + 5313), "flops": 3 * B * products}
        return {"bytes": 4 * 17 * B, "flops": B * products}
    n = case["N"] + 1
    E = len(mesh_of(case)[0])
    nodes = E * n * n
    if case["kind"] == "sensors":
        # the state three times (three calls), the outputs; two quantities' modes by x and y sums
        return {"bytes": 3 * 32 * nodes + 4 * E * 18, "flops": nodes * (5 * 4 * n + 30) + E * 2 * 5184}
    # a stage reads its input and (but for the first) the step's start and writes its
    # output; time step and download read the state once, the download writes it.
    # Operations of a node and stage: N pair fluxes of about 50, two logarithms,
    # two subcell fluxes, its share of the surface, the limiter
    stage = case["N"] * 50 + 60 + 80 + 4 * 70 // n + 250
    extra = {"local": 900, "lowsol": 700, "combined": 100}.get(case["limiter"], 0)
    return {"bytes": nodes * (case["steps"] * 288 + 64), "flops": nodes * case["steps"] * (3 * (stage + extra) + 40)}


# --------------------------------------------------------------------------
# the same in plain 64-bit arithmetic
# --------------------------------------------------------------------------
@functools.lru_cache(maxsize=4)
def operators(N):
    """LGL nodes and weights, 2Q - B, mortar interpolation and projection, the
    subcell overlaps across a mortar, and the nodal-to-modal transform."""
    L = np.polynomial.legendre
    n = N + 1
    x = np.concatenate([[-1.0], np.sort(L.legroots(L.legder([0] * N + [1])).real), [1.0]])
    V = L.legvander(x, N)
    w = 2.0 / (N * n * V[:, N] ** 2)
    D = np.stack([L.legval(x, L.legder(np.eye(n)[k])) for k in range(n)], axis=1) @ np.linalg.inv(V)
    S = 2 * w[:, None] * D
    S[0, 0] += 1
    S[N, N] -= 1
    lag = lambda s: L.legvander(s, N) @ np.linalg.inv(V)  # noqa: E731
    gx, gw = L.leggauss(n + 1)
    half = [(gx + h) / 2 for h in (-1, 1)]
    mass = lag(gx).T @ (gw[:, None] * lag(gx))
    inter = np.stack([lag((x + h) / 2) for h in (-1, 1)])
    proj = np.stack([np.linalg.solve(mass, 0.5 * lag(s).T @ (gw[:, None] * lag(gx))) for s in half])
    C = np.concatenate([[0.0], np.cumsum(w)])
    small = np.concatenate([-1 + C / 2, C[1:] / 2])  # edges of the 2n small subcells
    big = -1 + C
    over = np.minimum(big[1:, None], small[None, 1:]) - np.maximum(big[:-1, None], small[None, :-1])
    modal = np.linalg.inv(V * np.sqrt((2 * np.arange(n) + 1) / 2.0))
    dev = lambda a: torch.tensor(a, dtype=torch.float64, device="cuda")  # noqa: E731
    return x, dev(w), dev(S), dev(inter), dev(proj), dev(np.where(over > 1e-12, over, 0.0)), dev(modal)


class Plain:
    """Positivity-limited (or unlimited) SSP-RK3 steps on a periodic mesh."""

    def __init__(self, c):
        self.c, self.N, self.g = c, c["N"], GAMMA.get(c["flow"], 1.4)
        self.x, self.w, self.S, self.I, self.Pr, self.W, self.modal = operators(self.N)
        level, ix, iy = (a.astype(np.int64) for a in mesh_of(c))
        nx, ny = c["nx"], c["ny"]
        x0, y0, Lx, Ly = BOX[c["flow"]]
        hx, hy = Lx / (nx << level), Ly / (ny << level)
        t = 0.5 * (self.x + 1.0)
        X = np.broadcast_to(x0 + (ix[:, None, None] + t[None, None, :]) * hx[:, None, None], (len(level), c["N"] + 1, c["N"] + 1))
        Y = np.broadcast_to(y0 + (iy[:, None, None] + t[None, :, None]) * hy[:, None, None], X.shape)
        dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()  # noqa: E731
        self.X, self.Y, self.hx, self.hy = dev(X), dev(Y), dev(hx), dev(hy)
        key = lambda l, i, j: (l << 48) | ((i % (nx << l)) << 24) | (j % (ny << l))  # noqa: E731
        keys = key(level, ix, iy)
        order = np.argsort(keys)

        def find(l, i, j):
            k = key(np.maximum(l, 0), i, j)
            at = order[np.minimum(np.searchsorted(keys, k, sorter=order), len(keys) - 1)]
            return np.where((keys[at] == k) & (l >= 0), at, -1)

        self.near, self.mortars = [], []  # same-level neighbours; (face, large, small 0, small 1)
        for f, (dx, dy) in enumerate(((-1, 0), (1, 0), (0, -1), (0, 1))):
            same = find(level, ix + dx, iy + dy)
            self.near.append(dev(same))
            cx = 2 * ix + (dx < 0) * -1 + (dx > 0) * 2
            cy = 2 * iy + (dy < 0) * -1 + (dy > 0) * 2
            s0 = find(level + 1, cx, cy)
            s1 = find(level + 1, cx + (dx == 0), cy + (dy == 0))
            m = np.nonzero((same < 0) & (s0 >= 0) & (s1 >= 0))[0]
            if len(m):
                self.mortars.append((f, dev(m), dev(s0[m]), dev(s1[m])))

    def start(self, seed):
        return initial(self.c["flow"], self.X, self.Y, seed)

    def prim(self, u, ax=1):
        r, m1, m2, e = u.unbind(ax)
        v1, v2 = m1 / r, m2 / r
        p = (self.g - 1) * (e - 0.5 * (m1 * v1 + m2 * v2))
        return r, v1, v2, p, torch.sqrt(self.g * p / r)

    def speed(self, u, d, ax=1):
        q = self.prim(u, ax)
        return q[1 + d].abs() + q[4]

    def llf(self, ul, ur, d, ax=1):
        """Flux in the direction d from the low side ul to the high side ur."""
        def flux(u):
            r, v1, v2, p, _ = self.prim(u, ax)
            vn = (v1, v2)[d]
            m = list(u.unbind(ax))
            f = [m[0] * vn, m[1] * vn, m[2] * vn, (m[3] + p) * vn]
            f[1 + d] = f[1 + d] + p
            return torch.stack(f, ax)
        lam = torch.maximum(self.speed(ul, d, ax), self.speed(ur, d, ax)).unsqueeze(ax)
        return 0.5 * (flux(ul) + flux(ur)) - 0.5 * lam * (ur - ul)

    def pair(self, a, b, d):
        """The entropy-conserving two-point flux (Ranocha) between primitives a, b."""
        def lmean(p, q, inv):
            f2 = ((p - q) / (p + q)) ** 2
            ser = 1 + f2 * (1 / 3 + f2 * (1 / 5 + f2 * (1 / 7 + f2 * (1 / 9 + f2 / 11))))
            rough = f2 > 1e-3
            one = torch.ones_like(p)
            lg = torch.log(torch.where(rough, p / q, 2 * one)) / torch.where(rough, p - q, one)
            i = torch.where(rough, lg, 2 * ser / (p + q))
            return i if inv else 1 / i
        (ra, xa, ya, pa, _), (rb, xb, yb, pb, _) = a, b
        na, ta, nb, tb = (xa, ya, xb, yb) if d == 0 else (ya, xa, yb, xb)
        f0 = lmean(ra, rb, False) * 0.5 * (na + nb)
        fn = f0 * 0.5 * (na + nb) + 0.5 * (pa + pb)
        ft = f0 * 0.5 * (ta + tb)
        f3 = f0 * (0.5 * (na * nb + ta * tb) + lmean(ra / pa, rb / pb, True) / (self.g - 1)) + 0.5 * (pa * nb + pb * na)
        return torch.stack([f0, fn, ft, f3] if d == 0 else [f0, ft, fn, f3], 1)

    @staticmethod
    def trace(u, f):
        return (u[..., :, 0], u[..., :, -1], u[..., 0, :], u[..., -1, :])[f]

    def lines(self, u, d):
        """u with the positions along direction d last (d = 1: transposed)."""
        return u if d == 0 else u.transpose(-1, -2)

    def max_dt(self, u, cfl):
        s, n, h = torch.zeros_like(u[:, 0]), self.N + 1, (self.hx, self.hy)
        m = self.w[:, None] * self.w[None, :] * (self.hx * self.hy / 4)[:, None, None]
        for d in (0, 1):
            lam, acc = self.lines(self.speed(u, d), d), self.lines(s, d)
            edge = 0.5 * self.w[None, :, None] * h[1 - d][:, None, None] * torch.maximum(lam[..., 1:], lam[..., :-1])
            acc[..., 1:] += edge
            acc[..., :-1] += edge
        for f in range(4):
            d, nb = f // 2, self.near[f]
            lam, acc = self.speed(u, d), self.trace(s, f)
            other = self.trace(lam, f ^ 1)[nb.clamp(min=0)]
            e = 0.5 * self.w * h[1 - d][:, None] * torch.maximum(self.trace(lam, f), other)
            acc += torch.where(nb[:, None] >= 0, e, torch.zeros_like(e))
        for f, L, *sm in self.mortars:
            d = f // 2
            lam = self.speed(u, d)
            two = torch.cat([self.trace(lam, f ^ 1)[k] for k in sm], 1)
            e = 0.5 * self.W * h[1 - d][L][:, None, None] * torch.maximum(self.trace(lam, f)[L][:, :, None], two[:, None, :])
            self.trace(s, f).index_add_(0, L, e.sum(2))
            for k, part in zip(sm, e.sum(1).split(n, 1)):
                self.trace(s, f ^ 1).index_add_(0, k, part)
        return cfl / (s / m).max()

    def root(self, u, d, pt):
        """Largest theta in [0, 1] with a density above zero and a pressure of at
        least pt at u + theta d (quadratic in theta; u itself is inside)."""
        e0 = u[:, 3] - pt / (self.g - 1)
        g0 = u[:, 0] * e0 - 0.5 * (u[:, 1] ** 2 + u[:, 2] ** 2)
        g1 = d[:, 0] * e0 + u[:, 0] * d[:, 3] - u[:, 1] * d[:, 1] - u[:, 2] * d[:, 2]
        g2 = d[:, 0] * d[:, 3] - 0.5 * (d[:, 1] ** 2 + d[:, 2] ** 2)
        r1 = u[:, 0] + d[:, 0]
        full = (r1 > 0) & ((e0 + d[:, 3]) * r1 - 0.5 * ((u[:, 1] + d[:, 1]) ** 2 + (u[:, 2] + d[:, 2]) ** 2) >= 0)
        sq = torch.sqrt((g1 * g1 - 4 * g2 * g0).clamp(min=0))
        q = -0.5 * (g1 + torch.where(g1 >= 0, sq, -sq))
        th = torch.ones_like(g0)
        for t in (q / g2, g0 / q, torch.where(d[:, 0] < 0, -u[:, 0] / d[:, 0], th)):
            th = torch.where((t > 0) & (t < th), t, th)
        return torch.where((g0 > 0) & (u[:, 0] > 0), torch.where(full, torch.ones_like(th), th), torch.zeros_like(th))

    def euler(self, u, dt):
        """One limited forward-Euler step."""
        n, h, w, limit = self.N + 1, (self.hx, self.hy), self.w, self.c["limiter"] != "none"
        im = 1 / (w[:, None] * w[None, :] * (self.hx * self.hy / 4)[:, None, None])
        res, inc = torch.zeros_like(u), []
        prim = self.prim(u)
        for d in (0, 1):
            a, ul = [self.lines(q, d) for q in prim], self.lines(u, d)
            hs = 0.5 * h[1 - d][:, None, None, None]
            low = hs * self.llf(ul[..., :-1], ul[..., 1:], d)
            high = torch.zeros_like(low)
            for l in range(n):
                for k in range(l + 1, n):
                    high[..., l:k] += (hs[..., 0] * self.S[l, k] * self.pair([q[..., l] for q in a], [q[..., k] for q in a], d))[..., None]
            wl = w[None, None, :, None]
            r = self.lines(res, d)
            r[..., 1:] += wl * low
            r[..., :-1] -= wl * low
            inc.append(wl * (high - low))
        slots, count = [], torch.zeros_like(u[:, 0])
        for f in range(4):
            d, sg, nb = f // 2, -1.0 if f & 1 else 1.0, self.near[f]
            own, other = self.trace(u, f), self.trace(u, f ^ 1)[nb.clamp(min=0)]
            F = self.llf(own, other, d) if f & 1 else self.llf(other, own, d)
            F = sg * 0.5 * w * h[1 - d][:, None, None] * F
            self.trace(res, f).add_(torch.where(nb[:, None, None] >= 0, F, torch.zeros_like(F)))
        for f, L, *sm in self.mortars:
            d, sg = f // 2, -1.0 if f & 1 else 1.0
            hl = h[1 - d][L][:, None, None]
            big, two = self.trace(u, f)[L], [self.trace(u, f ^ 1)[k] for k in sm]
            flux = lambda a, b: self.llf(a, b, d) if f & 1 else self.llf(b, a, d)  # noqa: E731
            each = flux(big[..., :, None].expand(-1, -1, -1, 2 * n), torch.cat(two, 2)[..., None, :].expand(-1, -1, n, -1))
            each = sg * 0.5 * hl[..., None] * self.W * each
            lo_big, lo_two = each.sum(3), [-x for x in each.sum(2).split(n, 2)]
            inner = [big @ self.I[k].T for k in (0, 1)]
            hi = []
            for k in (0, 1):
                p = self.prim(inner[k])[3]
                fl = flux(inner[k], two[k])
                hi.append(torch.where(((inner[k][:, 0] > 0) & (p > 0))[:, None], fl, torch.full_like(fl, math.nan)))
            hi_big = sg * 0.5 * hl * w * (hi[0] @ self.Pr[0].T + hi[1] @ self.Pr[1].T)
            self.trace(res, f).index_add_(0, L, lo_big)
            self.trace(count, f).index_add_(0, L, torch.ones_like(big[:, 0]))
            sides = [(f, L, hi_big - lo_big)]
            for k in (0, 1):
                self.trace(res, f ^ 1).index_add_(0, sm[k], lo_two[k])
                self.trace(count, f ^ 1).index_add_(0, sm[k], torch.ones_like(big[:, 0]))
                sides.append((f ^ 1, sm[k], -sg * 0.25 * hl * w * hi[k] - lo_two[k]))
            slots.append(sides)
        low = u + dt * im[:, None] * res
        plow = self.prim(low)[3]
        rmin, pmin = 0.1 * low[:, 0], 0.1 * plow
        theta = torch.ones_like(rmin)
        faces = []  # per direction: the increments of the nodes on the low and the high side
        for d in (0, 1):
            i = dt * self.lines(im, d)[:, None]
            faces.append((-i[..., :-1] * inc[d], i[..., 1:] * inc[d]))
        if limit:
            neg = torch.zeros_like(rmin)
            for d in (0, 1):
                acc = self.lines(neg, d)
                acc[..., :-1] += faces[d][0][:, 0].clamp(max=0)
                acc[..., 1:] += faces[d][1][:, 0].clamp(max=0)
            z = ((rmin * (1 + 2.0 ** -40) - low[:, 0]) / neg).clamp(0, 1)
            theta = torch.where(neg < 0, z, theta)
            for d in (0, 1):
                lo, pt, th = self.lines(low, d), self.lines(pmin, d) * (1 + 2.0 ** -40), self.lines(theta, d)
                r0 = self.root(lo[..., :-1], 4 * faces[d][0], pt[..., :-1])
                r1 = self.root(lo[..., 1:], 4 * faces[d][1], pt[..., 1:])
                th[..., :-1] = torch.minimum(th[..., :-1], r0)
                th[..., 1:] = torch.minimum(th[..., 1:], r1)
        vol = low.clone()
        for d in (0, 1):
            th, v = self.lines(theta, d), self.lines(vol, d)
            t = torch.minimum(th[..., :-1], th[..., 1:])[:, None]
            v[..., :-1] += t * faces[d][0]
            v[..., 1:] += t * faces[d][1]
        out = vol.clone()
        for sides in slots:
            ts, incs = None, []
            for f, e, dS in sides:
                c = dt * self.trace(im, f)[e][:, None] * dS
                incs.append(c)
                dc = self.trace(count, f)[e][:, None] * c
                v, r0, p0 = self.trace(vol, f)[e], self.trace(rmin, f)[e], self.trace(pmin, f)[e]
                z = ((r0 * (1 + 2.0 ** -41) - v[:, 0]) / dc[:, 0]).clamp(min=0)
                t = torch.minimum(torch.where((dc[:, 0] < 0) & (z < 1), z, torch.ones_like(z)),
                                  self.root(v, dc, p0 * (1 + 2.0 ** -41)))
                t = torch.where(torch.isfinite(dc).all(1), t, torch.zeros_like(t)) if limit else torch.ones_like(t)
                ts = t.amin(1) if ts is None else torch.minimum(ts, t.amin(1))
            for (f, e, _), c in zip(sides, incs):
                self.trace(out, f).index_add_(0, e, torch.where((ts > 0)[:, None, None], ts[:, None, None] * c, torch.zeros_like(c)))
        return out

    def step(self, u, cfl):
        dt = self.max_dt(u, cfl)
        v = self.euler(u, dt)
        v = 0.75 * u + 0.25 * self.euler(v, dt)
        return u / 3 + 2 / 3 * self.euler(v, dt), float(dt)


def network(w, x, rounded):
    """The network with the parameters w (rounded to 16 bits, as it is defined)."""
    if rounded:
        w = w.float().bfloat16().double()
    W1, b1, W2, b2, W3, b3 = w.split([1024, 64, 4096, 64, 64, 1])
    z = torch.relu(x @ W1.reshape(64, 16).T + b1)
    return torch.relu(z @ W2.reshape(64, 64).T + b2) @ W3 + b3


def exact(case, seed):
    if case["kind"] in ("train", "network"):
        x, t = batch_of(case, seed)
        w = torch.from_numpy(weights_of(seed)).cuda().bfloat16().double().requires_grad_(True)
        y = network(w, x.double(), False)
        if case["kind"] == "network":
            return {"y": y.detach()}
        loss = ((y - t.double()) ** 2).mean()
        loss.backward()
        return {"grad": w.grad, "loss": float(loss)}
    # adapted meshes, boundaries and the limiters that search their factors by
    # iteration have no plain form here
    if case["kind"] == "adapt" or case["flow"] in ("jet", "dmr") or case.get("limiter", "none") not in ("none", "positivity"):
        return None
    if case["kind"] == "sensors":
        m = Plain(dict(case, limiter="positivity"))
        u = m.start(seed)
        for _ in range(3):
            u, _ = m.step(u, 0.5)
        N, V = case["N"], m.modal
        r, _, _, p, _ = m.prim(u)
        modes = lambda q: (torch.einsum("ia,jb,eba->eji", V, V, q)) ** 2  # noqa: E731
        feat = []
        for q in (modes(r), modes(p)):
            all_ = q.sum((1, 2))[:, None]
            feat += [q.sum(1)[:, N - 3:] / all_, q.sum(2)[:, N - 3:] / all_]
        q = modes(r * p)
        full, l1, l2 = q.sum((1, 2)), q[:, :N, :N].sum((1, 2)), q[:, :N - 1, :N - 1].sum((1, 2))
        en = torch.maximum((full - l1) / full, (l1 - l2) / l1)
        T = 0.5 * 10.0 ** (-1.8 * (N + 1) ** 0.25)
        al = 1 / (1 + torch.exp(-math.log((1 - 1e-4) / 1e-4) / T * (en - T)))
        al = torch.where(al < 1e-3, torch.zeros_like(al), al).clamp(max=0.5)
        feat = torch.cat(feat, 1)
        return {"features": feat, "modal": al,
                "learned": network(torch.from_numpy(weights_of(seed)).cuda().double(), feat, True)}
    m = Plain(case)
    u, said = m.start(seed), []
    for _ in range(case["steps"]):
        u, dt = m.step(u, case["cfl"])
        said.append({"dt": dt, "violations": None, "fv_inadmissible": None})
    return {"stats": said if case["loop"] != "plain" else [], "u": u}
