"""Performance cases of the interface solver: the calls that a mesh-generation program makes, with their inputs.

A case names one entry point of the package (or the short sequence of them
that makes up a mesh step), the sub-domain layout it runs on and its sizes.
``listed()`` holds the sizes of the repository's own workloads -- the paper's
41 x 41 run, the 768-cell run, the moving bump with 1521 nodes, the network's
training -- and ``draw()`` more of the same ranges.

Inputs are synthetic and come from the seed alone: the time at which the
density is frozen (or the path's time origin), the Philox seed, the mesh that
the step starts from, the network's weights and the training labels.
"""
from __future__ import annotations

import math
import random

import numpy as np
import torch

import paper_1402_0266_amd as fk
from paper_1402_0266_amd.mesh_run import Density, GridData, interface_nodes

DEV = "cuda"
BUMP, MOVING, TWO, RING = 1, 2, 3, 4
BACKWARD, FROZEN = 0, 1
IDENTITY, GRID, EQUIDISTRIBUTED = 0, 3, 4
UNCLAMPED, EXTEND, BRIDGE = 0, 2, 3


# ---------------------------------------------------------------------------
# Cases
# ---------------------------------------------------------------------------
def listed():
    return [
        # one mesh step's interface solve of the paper's run: 77 nodes, 20 sub-steps, the smallest call of a run
        dict(name="interface_ring_77", call="interface", density="ring", px=2, m=20, t=1e-3, steps=20, paths=10000),
        # the same step of the 768-cell run: 10689 nodes
        dict(name="interface_two_bumps_10689", call="interface", density="two", px=8, m=96, t=5e-4, steps=20,
             paths=16384),
        # a time-dependent density from the uniform mesh over a long horizon (10^4 steps): the headline workload's
        # nodes and steps, at a path count of about an eighteenth of what RMS 1e-3 takes
        dict(name="interface_moving_1521", call="interface", density="moving", px=4, m=64, t=0.1, steps=10000,
             paths=4096),
        # several time levels with layouts of their own in one launch
        dict(name="batch_16_levels", call="batch", density="moving", levels=16, cells=128, t=0.16, steps=1600,
             paths=1024),
        # interface values of the steady mesh: paths run until they leave the square, found by the bridge test
        dict(name="interface_steady_125", call="steady", density="bump", px=2, m=32, t=3.0, steps=30000, paths=16384),
        # the mesh step with the mesh's own gradient as control
        dict(name="cv_mesh_10689", call="cv_mesh", density="two", px=8, m=96, t=5e-4, steps=20, paths=16384, stride=2),
        # the network as control, Dynkin form, at the path count that RMS 1e-3 takes with it
        dict(name="cv_dynkin_1521", call="cv_net", form="dynkin", density="moving", px=4, m=64, t=0.1, steps=10000,
             paths=173, stride=100, precision="split"),
        # ... martingale form, gradient rounded to BF16, as the short fit uses it
        dict(name="cv_martingale_1521", call="cv_net", form="martingale", density="moving", px=4, m=64, t=0.1,
             steps=10000, paths=696, stride=500, precision="bf16"),
        # Adam steps of the network's fit
        dict(name="train_200", call="train", labels=200772, steps=200, batch=8192),
        # the sub-domain solves of the paper's run and of the 768-cell run
        dict(name="subdomain_ring_41", call="subdomain", density="ring", px=2, py=2, cells=40, edges="equidistributed",
             steady=False),
        dict(name="subdomain_two_bumps_769", call="subdomain", density="two", px=8, py=8, cells=768, edges="identity",
             steady=False),
        # a whole step of the paper's run: interface solve, sub-domain solves, mesh quality
        dict(name="mesh_step_ring_41", call="mesh_step", density="ring", px=2, m=20, t=1e-3, steps=20, paths=10000,
             keys=False),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng: random.Random):
    call = rng.choice(["interface", "interface", "long", "batch", "steady", "cv_mesh", "cv_net", "train", "subdomain",
                       "subdomain", "mesh_step"])
    if call in ("interface", "cv_mesh", "mesh_step"):
        density = rng.choice(["ring", "two", "moving"])
        px, m = rng.randint(2, 8), _log(rng, 16, 96)
        # the path steps of the 768-cell run are the most
        most = 3.5e9 / (20 * fk.n_interface_nodes(px, m))
        steps = rng.choice([8, 19, 20, 20, 32])
        paths = min(_log(rng, 1000, 16384), int(most * 20 / steps))
        c = dict(call=call, density=density, px=px, m=m, t=rng.choice([5e-4, 1e-3]), steps=steps, paths=paths)
        if call == "cv_mesh":
            c["stride"] = rng.choice([2, 4, 20])
        if call == "mesh_step":
            c["keys"] = rng.random() < 0.5
        return c
    if call == "long":
        px, m = rng.randint(2, 4), _log(rng, 8, 64)
        steps = _log(rng, 500, 10000)
        most = 2e10 / (steps * 0.37 * fk.n_interface_nodes(px, m))
        return dict(call="interface", density=rng.choice(["bump", "moving"]), px=px, m=m, t=rng.choice([0.05, 0.1]),
                    steps=steps, paths=max(64, min(_log(rng, 256, 20000), int(most))))
    if call == "batch":
        return dict(call="batch", density="moving", levels=rng.randint(2, 16), cells=rng.choice([32, 60, 96, 128]), t=0.16,
                    steps=_log(rng, 200, 1600), paths=_log(rng, 100, 1024))
    if call == "steady":
        return dict(call="steady", density=rng.choice(["bump", "ring"]), px=2, m=rng.randint(14, 32), t=3.0,
                    steps=30000, paths=_log(rng, 1000, 16384))
    if call == "cv_net":
        form = rng.choice(["dynkin", "martingale"])
        c = dict(call="cv_net", form=form, density="moving", px=rng.randint(2, 4), m=_log(rng, 16, 64), t=0.1,
                 steps=_log(rng, 1000, 10000), paths=_log(rng, 100, 600), stride=rng.choice([20, 100, 200, 500]),
                 precision="split" if form == "dynkin" else rng.choice(["split", "bf16"]))
        c["paths"] = max(64, min(c["paths"], int(c["paths"] * 8e11 / work(c)["flops"])))
        return c
    if call == "train":
        return dict(call="train", labels=_log(rng, 10000, 200000), steps=_log(rng, 20, 200), batch=_log(rng, 500, 8192))
    px, py = rng.randint(1, 8), rng.randint(1, 8)
    side = math.lcm(px, py) * 2
    # whole sub-domains of at least 5 and at most 96 cells a side
    lo, hi = -(-5 * max(px, py) // side), 96 * min(px, py) // side
    cells = side * _log(rng, max(1, lo), max(1, lo, hi))
    if min(cells // px, cells // py) > 96 or max(cells // px, cells // py) > 192 or cells > 768:
        return draw(rng)
    density = rng.choice(["bump", "two", "ring"])
    if cells < {"bump": 32, "two": 64, "ring": 16}[density]:   # the grid has to resolve the density
        return draw(rng)
    return dict(call="subdomain", density=density, px=px, py=py, cells=cells,
                edges=rng.choice(["identity", "equidistributed"]), steady=rng.random() < 0.25)


# ---------------------------------------------------------------------------
# Inputs
# ---------------------------------------------------------------------------
def _density(name, mode, t_freeze):
    w = 2.0 * math.pi
    if name == "bump":
        return Density(BUMP, BACKWARD, 10.0, 0.01, 0.3, 0.6, 0.0, 0.0, 0.0)
    if name == "moving":
        return Density(MOVING, mode, 20.0, 0.005, 0.5, 0.5, 0.25, w, t_freeze)
    if name == "two":
        return Density(TWO, mode, 30.0, 0.003, 0.5, 0.5, 0.25, w, t_freeze)
    return Density(RING, mode, 10.0, -50.0, 0.5, 0.5, 0.25, w, t_freeze)


def _scalars(seed):
    """(time of the density, Philox seed) of a seed."""
    r = np.random.default_rng([int(seed), 1])
    return float(r.uniform(0.05, 0.75)), int(r.integers(1, 1 << 40))


def _mesh(cells, seed):
    """A smooth invertible map with the identity on the edges: the mesh a step starts from."""
    r = np.random.default_rng([int(seed), 2])
    x = torch.arange(cells + 1, dtype=torch.float64, device=DEV) / cells
    out = []
    for comp in range(2):
        v = x.repeat(cells + 1, 1) if comp == 0 else x[:, None].repeat(1, cells + 1)
        for a in (1, 2, 3):
            for b in (1, 2, 3):
                v = v + float(r.uniform(-0.04, 0.04)) / (a * b) * torch.sin(a * math.pi * x)[None, :] * torch.sin(
                    b * math.pi * x)[:, None]
        out.append(v.contiguous())
    return out


def _iface(px, py, cells, xi, eta):
    """The mesh's values at the interface nodes of px x py sub-domains, in the solve's order."""
    mx, my = cells // px, cells // py
    ij = [(a * mx, j) for a in range(1, px) for j in range(1, cells)]
    ij += [(i, c * my) for c in range(1, py) for i in range(1, cells) if i % mx]
    ij = torch.tensor(ij, dtype=torch.int64, device=DEV).reshape(-1, 2)
    return xi[ij[:, 1], ij[:, 0]].contiguous(), eta[ij[:, 1], ij[:, 0]].contiguous()


def _weights(seed):
    """Glorot-uniform weights, zero biases, in the network's parameter order."""
    r = np.random.default_rng([int(seed), 3])
    out = []
    for shape in [(64, 3), (64,), (64, 64), (64,), (64, 64), (64,), (2, 64), (2,)]:
        a = math.sqrt(6.0 / sum(shape)) if len(shape) == 2 else 0.0
        out.append(r.uniform(-a, a, size=shape).astype(np.float32).ravel())
    return np.concatenate(out)


def _rows(n, *names):
    out = {k: torch.empty(n, dtype=torch.float64, device=DEV) for k in names}
    out["total_steps"] = torch.zeros(1, dtype=torch.int64, device=DEV)
    return out


def _levels(case):
    """(density, t, t_init, nodes, level id) of each level of a batch: a layout drawn for each level."""
    r = np.random.default_rng([case["cells"], case["levels"]])
    dens, out = _density(case["density"], BACKWARD, 0.0), []
    for k in range(1, case["levels"] + 1):
        fit = [p for p in range(2, 9) if case["cells"] % p == 0]
        px = int(r.choice(fit))
        out.append((dens, case["t"] * k / case["levels"], 0.0, interface_nodes(px, case["cells"] // px), k))
    return out


def prepare(case, seed):
    call = case["call"]
    t_n, key = _scalars(seed)
    s = dict(case=case, key=key, t_n=t_n)
    if call == "train":
        r = np.random.default_rng([int(seed), 5])
        n = case["labels"]
        txy = r.uniform(0.0, 1.0, size=(n, 3)).astype(np.float32)
        txy[:, 0] *= 0.1
        s["txy"] = torch.from_numpy(txy).to(DEV)
        t, x, y = (s["txy"][:, i].double() for i in range(3))
        cx, cy = 0.5 + 0.25 * torch.cos(2 * math.pi * (t + t_n)), 0.5 + 0.25 * torch.sin(2 * math.pi * (t + t_n))
        e = torch.exp(-((x - cx) ** 2 + (y - cy) ** 2) / 0.02) * torch.sin(math.pi * x) * torch.sin(math.pi * y)
        noise = torch.from_numpy(r.normal(0.0, 0.003, size=(n, 2))).to(DEV)   # the labels' Monte-Carlo error
        s["target"] = (torch.stack([x + (x - cx) * e, y + (y - cy) * e], 1) + noise).float().contiguous()
        s["cv"] = fk.FkCv(_weights(seed), t_scale=0.1, identity_base=True)
        return s
    if call == "batch":
        s["batch"] = fk.FkBatch(_levels(case), GridData(t_init=0.0, init_kind=IDENTITY, score_mode=UNCLAMPED),
                                case["t"] / case["steps"], case["paths"], seed=key, device=DEV)
        s["out"] = s["batch"].outputs()
        return s
    if call == "subdomain":
        N = case["cells"]
        s["density"] = _density(case["density"], FROZEN, t_n)
        s["xi"], s["eta"] = _mesh(N, seed)
        s["iface"] = _iface(case["px"], case["py"], N, s["xi"], s["eta"])
        s["out"] = tuple(torch.empty_like(s["xi"]) for _ in range(2))
        need = fk.subdomain_workspace_bytes_rect(case["px"], case["py"], N)
        s["workspace"] = torch.empty(max(need, 256), dtype=torch.uint8, device=DEV)
        return s
    px, m, n_paths = case["px"], case["m"], case["paths"]
    N = px * m
    nodes = interface_nodes(px, m)
    n = len(nodes)
    s["pts"] = torch.tensor(nodes, dtype=torch.float64, device=DEV)
    s["dt"] = case["t"] / case["steps"]
    short = case["steps"] <= 64
    s["density"] = _density(case["density"], FROZEN if short or call == "steady" else BACKWARD, t_n)
    s["grids"] = None
    if call == "steady":
        # the uniform mesh, whose edge nodes hold the boundary data
        x = torch.arange(N + 1, dtype=torch.float64, device=DEV) / N
        s["grids"] = (x.repeat(N + 1, 1).contiguous().view(-1), x[:, None].repeat(1, N + 1).contiguous().view(-1))
        s["data"] = GridData(t_init=0.0, bdry_kind=GRID, score_mode=BRIDGE)
    elif short:
        s["xi"], s["eta"] = _mesh(N, seed)
        s["grids"] = (s["xi"].view(-1), s["eta"].view(-1))
        s["data"] = GridData(t_init=t_n, score_mode=EXTEND)
    else:
        s["data"] = GridData(t_init=0.0 if call == "cv_net" else t_n, init_kind=IDENTITY, score_mode=UNCLAMPED)
    s["out"] = _rows(n, "xi", "eta", "se_xi", "se_eta")
    need = fk.fk_interface_workspace_bytes(n, n_paths)
    if call == "cv_mesh":
        need = fk.fk_interface_cv_grid_workspace_bytes(n, n_paths, N)
    elif call == "cv_net":
        s["cv"] = fk.FkCv(_weights(seed), t_scale=0.1, identity_base=True, grad_precision=case["precision"])
        need = int(fk.library().fk_interface_cv_workspace_bytes(n, n_paths))
    s["workspace"] = torch.empty(max(need, 256), dtype=torch.uint8, device=DEV)
    if call == "mesh_step":
        s["new"] = (torch.empty_like(s["xi"]), torch.empty_like(s["eta"]))
        s["sub_workspace"] = torch.empty(max(fk.subdomain_workspace_bytes(px, m), 256), dtype=torch.uint8, device=DEV)
        s["quality"] = torch.empty(2, dtype=torch.float64, device=DEV)
        if case["keys"]:
            s["wg"] = torch.empty((N + 1, N + 1), dtype=torch.float64, device=DEV)
            s["wb"] = torch.empty((N + 1, N + 1, 2), dtype=torch.float32, device=DEV)
            s["mask"] = torch.empty(n, dtype=torch.uint8, device=DEV)
            s["bdry_ws"] = torch.empty(max(fk.fk_boundary_workspace_bytes(N), 256), dtype=torch.uint8, device=DEV)
    return s


# ---------------------------------------------------------------------------
# One pass
# ---------------------------------------------------------------------------
def _edges(case):
    return EQUIDISTRIBUTED if case.get("edges") == "equidistributed" or case["density"] == "ring" else IDENTITY


def _estimates(out):
    return {k: v for k, v in out.items() if not k.startswith("_")}


def run(s):
    case = s["case"]
    call = case["call"]
    if call == "train":
        loss = s["cv"].train(s["txy"], s["target"], steps=case["steps"], batch=case["batch"], lr=1e-3, seed=s["key"])
        return {"loss": loss, "weights": s["cv"].params()[0]}
    if call == "batch":
        return _estimates(s["batch"].run(s["out"]))
    if call == "subdomain":
        edges = EQUIDISTRIBUTED if case["edges"] == "equidistributed" else IDENTITY
        dt = math.inf if case["steady"] else 5e-4
        return fk.subdomain_solve_rect(s["density"], s["t_n"], dt, case["px"], case["py"], case["cells"],
                                       None if case["steady"] else s["xi"], None if case["steady"] else s["eta"],
                                       *s["iface"], bdry_kind=edges, out=s["out"], workspace=s["workspace"])
    if call == "cv_mesh":
        return _estimates(fk.fk_interface_solve_cv(
            s["density"], s["data"], s["pts"], case["t"], s["dt"], case["paths"], None, stride=case["stride"],
            seed=s["key"], level_id=3, form=fk.FK_CV_MARTINGALE_GRID, plain=False, workspace=s["workspace"],
            grids=s["grids"], out=s["out"]))
    if call == "cv_net":
        form = fk.FK_CV_DYNKIN if case["form"] == "dynkin" else fk.FK_CV_MARTINGALE
        return _estimates(fk.fk_interface_solve_cv(
            s["density"], s["data"], s["pts"], case["t"], s["dt"], case["paths"], s["cv"], stride=case["stride"],
            seed=s["key"], form=form, plain=False, workspace=s["workspace"], out=s["out"]))
    if call == "mesh_step":
        return _mesh_step(s, case)
    return _estimates(fk.fk_interface_solve(s["density"], s["data"], s["pts"], case["t"], s["dt"], case["paths"],
                                            seed=s["key"], level_id=3, workspace=s["workspace"], grids=s["grids"],
                                            out=s["out"]))


def _mesh_step(s, case):
    """A mesh step as the run's driver makes it (Sect. 4), with all interface nodes or the key points only."""
    px, m, N, t_n, out = case["px"], case["m"], case["px"] * case["m"], s["t_n"], s["out"]
    dens, mask = s["density"], None
    if case["keys"]:
        fk.fk_density_sample(dens, t_n, N, out=s["wg"])
        dens = fk.GridDensity(s["wg"], grid_b=s["wb"])
        mask = fk.fk_key_points(s["wg"], px, m, out=s["mask"])
    fk.fk_interface_solve(dens, s["data"], s["pts"], case["t"], s["dt"], case["paths"], seed=s["key"], level_id=3,
                          workspace=s["workspace"], grids=s["grids"], out=out, mask=mask)
    if case["keys"]:
        fk.fk_boundary_data(dens, t_n, N, _edges(case), *s["new"], workspace=s["bdry_ws"])
        fk.fk_interface_interpolate_mask(px, m, mask, *s["new"], out["xi"], out["eta"])
    xi, eta = fk.subdomain_solve(dens, t_n, case["t"], px, m, s["xi"], s["eta"], out["xi"], out["eta"],
                                 bdry_kind=_edges(case), out=s["new"], workspace=s["sub_workspace"])
    fk.fk_mesh_quality(xi, eta, out=s["quality"])
    return {"iface_xi": out["xi"], "iface_eta": out["eta"], "xi": xi, "eta": eta, "quality": s["quality"]}


# ---------------------------------------------------------------------------
# What a pass cannot do without
# ---------------------------------------------------------------------------
def _path_steps(nodes, t, steps, paths):
    """Expected Euler-Maruyama steps: a proxy of each node's mean exit time, cut at the horizon."""
    ax, ay = nodes[:, 0] * (1 - nodes[:, 0]), nodes[:, 1] * (1 - nodes[:, 1])
    tau = 1.0 / (2.0 / ax + 2.0 / ay)
    return float(np.sum(tau * -np.expm1(-t / tau))) * steps / t * paths


def _sub_work(px, py, N):
    """Band LU of every sub-domain is not needed: a nested-dissection factorisation of an n = q x q grid takes about
    10 n^1.5 multiply-adds."""
    n = (N // px - 1) * (N // py - 1)
    return px * py * 2.0 * 10.0 * n ** 1.5, 8.0 * 4 * (N + 1) ** 2


def work(case):
    call = case["call"]
    if call == "train":
        # forward 2 P, backward 4 P operations a sample (P = 8706 weights)
        per = case["steps"] * case["batch"]
        return {"bytes": per * 20.0 + case["steps"] * 8706 * 4.0 * 6, "flops": per * 6.0 * 8706}
    if call == "subdomain":
        f, b = _sub_work(case["px"], case["py"], case["cells"])
        return {"bytes": b, "flops": f}
    if call == "batch":
        n, steps = 0, 0.0
        for _, t, _, p, _ in _levels(case):
            n += len(p)
            steps += _path_steps(p, t, case["steps"] * t / case["t"], case["paths"])
        return {"bytes": n * 48.0, "flops": 36.0 * steps}
    nodes = interface_nodes(case["px"], case["m"])
    # 36 operations a step: position, drift, Box-Muller, exit test
    steps = _path_steps(nodes, case["t"], case["steps"], case["paths"])
    flops, byt = 36.0 * steps, len(nodes) * 48.0
    N = case["px"] * case["m"]
    if call == "cv_mesh":
        flops += steps / case["stride"] * 20.0
        byt += 16.0 * (N + 1) ** 2
    if call == "cv_net":
        # two 64 x 64 hidden layers for each channel, at every evaluation point
        flops += steps / case["stride"] * (5 if case["form"] == "dynkin" else 3) * 2 * 2 * 4096.0
    if call == "mesh_step":
        f, b = _sub_work(case["px"], case["px"], N)
        flops, byt = flops + f, byt + b
    return {"bytes": byt, "flops": flops}


# ---------------------------------------------------------------------------
# The same results in 64 bits
# ---------------------------------------------------------------------------
def _philox(c0, c1, c2, c3, key):
    """Philox4x32-10 words of int64 tensors (Salmon et al., SC'11)."""
    M, k0, k1 = 0xFFFFFFFF, key & 0xFFFFFFFF, (key >> 32) & 0xFFFFFFFF
    for _ in range(10):
        p0, p1 = c0 * 0xD2511F53, c2 * 0xCD9E8D57
        c0, c1, c2, c3 = ((p1 >> 32) & M) ^ c1 ^ k0, p1 & M, ((p0 >> 32) & M) ^ c3 ^ k1, p0 & M
        k0, k1 = (k0 + 0x9E3779B9) & M, (k1 + 0xBB67AE85) & M
    return c0, c1, c2, c3


def _drift(d, tau, x, y):
    """-grad w / w at (x, y), the centre on its orbit at time tau."""
    moving = d.kind != BUMP
    ox, oy = (d.orbit_r * math.cos(d.omega * tau), d.orbit_r * math.sin(d.omega * tau)) if moving else (0.0, 0.0)
    dx, dy = x - (d.cx + ox), y - (d.cy + oy)
    if d.kind == RING:
        q = dx * dx + dy * dy - 0.01
        e = torch.exp(d.width2 * q.abs())
        f = 2.0 * d.amp * d.width2 * torch.sign(q) * e / (1.0 + d.amp * e)
        return f * dx, f * dy
    e1 = torch.exp(-(dx * dx + dy * dy) / d.width2)
    if d.kind == TWO:
        d2 = x - (d.cx - ox)
        e2 = torch.exp(-(d2 * d2 + dy * dy) / d.width2)
        f = 2.0 * d.amp / d.width2 / (1.0 + d.amp * (e1 + e2))
        return f * (e1 * dx + e2 * d2), f * (e1 + e2) * dy
    f = 2.0 * d.amp / d.width2 * e1 / (1.0 + d.amp * e1)
    return f * dx, f * dy


def _cell(x, y, n):
    i = torch.clamp(torch.floor(x * n), 0, n - 1).long()
    j = torch.clamp(torch.floor(y * n), 0, n - 1).long()
    return j * (n + 1) + i, x * n - i, y * n - j


def _bilinear(g, x, y, n, gradient=False):
    c, ax, ay = _cell(x, y, n)
    a, b, p, q = g[c], g[c + 1], g[c + n + 1], g[c + n + 2]
    if gradient:
        return n * ((b - a) + ay * ((q - p) - (b - a))), n * ((p - a) + ax * ((q - b) - (p - a)))
    return (1 - ay) * ((1 - ax) * a + ax * b) + ay * ((1 - ax) * p + ax * q)


def _simulate(dens, data, pts, t, dt, paths, key, level, grids=None, stride=0):
    """Means and standard errors of the Monte-Carlo estimate at pts, path by path in 64 bits."""
    K = math.ceil(t / dt - 1e-9)
    n_grid = int(round(grids[0].numel() ** 0.5)) - 1 if grids is not None else 0
    res = []
    per = max(1, (1 << 24) // paths)
    for a in range(0, len(pts), per):
        P = pts[a:a + per]
        nid = torch.arange(a, a + len(P), device=DEV).repeat_interleave(paths)
        path = torch.arange(paths, device=DEV).repeat(len(P))
        x, y = P[:, 0].repeat_interleave(paths), P[:, 1].repeat_interleave(paths)
        alive = torch.ones_like(x, dtype=torch.bool)
        zero = torch.zeros_like(x)
        mx, my, bx_, by_ = zero.clone(), zero.clone(), zero.clone(), zero.clone()
        G = None
        for k in range(K):
            if k % 2 == 0:
                words = _philox(torch.full_like(nid, k // 2), path, nid, torch.full_like(nid, level << 4), key)
                if stride and k % stride == 0:
                    if G is not None:
                        mx, my = mx + G[0] * bx_ + G[1] * by_, my + G[2] * bx_ + G[3] * by_
                    new = _bilinear(grids[0], x, y, n_grid, True) + _bilinear(grids[1], x, y, n_grid, True)
                    G = new if G is None else tuple(torch.where(alive, u, v) for u, v in zip(new, G))
                    bx_, by_ = zero.clone(), zero.clone()
            ra, rb = words[2 * (k % 2)], words[2 * (k % 2) + 1]
            D = dt if k < K - 1 else t - (K - 1) * dt
            u1 = 1.0 - (ra & 0x7FFFFF).double() * 2.0 ** -23
            rad, ang = torch.sqrt(-4.0 * D * torch.log(u1)), 2.0 * math.pi * 2.0 ** -23 * (rb & 0x7FFFFF).double()
            wx, wy = rad * torch.cos(ang), rad * torch.sin(ang)
            bx, by = _drift(dens, dens.t_freeze if dens.time_mode == FROZEN else data.t_init + t - k * dt, x, y)
            x, y = torch.where(alive, x + bx * D + wx, x), torch.where(alive, y + by * D + wy, y)
            bx_, by_ = torch.where(alive, bx_ + wx, bx_), torch.where(alive, by_ + wy, by_)
            alive &= (x >= 0) & (x <= 1) & (y >= 0) & (y <= 1)
        if data.init_kind == GRID:   # exits are scored with the mesh continued past its edge
            sx, sy = _bilinear(grids[0], x, y, n_grid), _bilinear(grids[1], x, y, n_grid)
        else:
            sx, sy = x, y
        if stride:
            sx, sy = sx - (mx + G[0] * bx_ + G[1] * by_), sy - (my + G[2] * bx_ + G[3] * by_)
        sx, sy = sx.view(len(P), paths), sy.view(len(P), paths)
        res.append(torch.stack([sx.mean(1), sy.mean(1), (sx.var(1) / paths).sqrt(), (sy.var(1) / paths).sqrt()]))
    r = torch.cat(res, 1)
    return {"xi": r[0], "eta": r[1], "se_xi": r[2], "se_eta": r[3], "total_steps": None}


def _density_value(d, t, x, y):
    moving = d.kind != BUMP
    ox, oy = (d.orbit_r * math.cos(d.omega * t), d.orbit_r * math.sin(d.omega * t)) if moving else (0.0, 0.0)
    r1 = (x - (d.cx + ox)) ** 2 + (y - (d.cy + oy)) ** 2
    if d.kind == RING:
        return 1.0 / (1.0 + d.amp * np.exp(d.width2 * np.abs(r1 - 0.01)))
    w = np.exp(-r1 / d.width2)
    if d.kind == TWO:
        w = w + np.exp(-((x - (d.cx - ox)) ** 2 + (y - (d.cy + oy)) ** 2) / d.width2)
    return 1.0 + d.amp * w


def _subdomains(dens, t_w, dt, px, py, N, xi, eta, iface, edges):
    """Backward-Euler (dt = inf: steady) solves of every sub-domain: block elimination by grid rows, dense blocks."""
    h, M = 1.0 / N, N + 1
    s = np.arange(M) / N
    out = [np.zeros((M, M)), np.zeros((M, M))]
    for comp in range(2):
        for e in range(2):
            out[comp][:, -e] = s if comp else float(e)      # the left and right edge
            out[comp][-e, :] = float(e) if comp else s      # the bottom and top edge
            if edges == EQUIDISTRIBUTED:
                g = 4096
                u = np.arange(N * g + 1) / (N * g)
                w = _density_value(dens, t_w, *((u, float(e)) if comp == 0 else (float(e), u)))
                cells = (w[:-1].reshape(N, g).sum(1) + 0.5 * (w[g::g] - w[:-1:g])) / (N * g)
                f = np.concatenate([[0.0], np.cumsum(cells)]) / cells.sum()
                if comp == 0:
                    out[0][-e, :] = f
                else:
                    out[1][:, -e] = f
    mx, my = N // px, N // py
    ij = [(a * mx, j) for a in range(1, px) for j in range(1, N)]
    ij += [(i, c * my) for c in range(1, py) for i in range(1, N) if i % mx]
    ij = np.array(ij, dtype=np.int64).reshape(-1, 2)
    for o, v in zip(out, iface):
        o[ij[:, 1], ij[:, 0]] = v
    X, Y = torch.from_numpy(np.tile(s, (M, 1))), torch.from_numpy(np.tile(s[:, None], (1, M)))
    bx, by = (v.numpy() for v in _drift(dens, t_w, X, Y))
    steady = math.isinf(dt)
    c, hd, diag = (1.0, 0.5 * h, 4.0) if steady else (dt / h ** 2, dt / (2 * h), 1.0 + 4.0 * dt / h ** 2)
    E, W, Nn, S = -c - hd * bx, -c + hd * bx, -c - hd * by, -c + hd * by
    q, rows = mx - 1, my - 1

    def part(g, j, di=0, dj=0):   # row j of every sub-domain's interior, [sub-domains, q]
        return np.stack([g[b * my + 1 + j + dj, a * mx + 1 + di:a * mx + 1 + di + q] for b in range(py) for a in range(px)])

    U, V = [], []
    for j in range(rows):
        T = np.zeros((px * py, q, q))
        idx = np.arange(q)
        T[:, idx, idx] = diag
        T[:, idx[:-1], idx[1:]] = part(E, j)[:, :-1]
        T[:, idx[1:], idx[:-1]] = part(W, j)[:, 1:]
        rhs = np.zeros((px * py, q, 2))
        for comp in range(2):
            r = np.zeros((px * py, q)) if steady else part((xi, eta)[comp], j).copy()
            r[:, -1] -= part(E, j)[:, -1] * part(out[comp], j, 1)[:, -1]
            r[:, 0] -= part(W, j)[:, 0] * part(out[comp], j, -1)[:, 0]
            if j == rows - 1:
                r -= part(Nn, j) * part(out[comp], j, 0, 1)
            if j == 0:
                r -= part(S, j) * part(out[comp], j, 0, -1)
            rhs[:, :, comp] = r
        if j:
            low = part(S, j)[:, :, None]
            T -= low * U[-1]
            rhs -= low * V[-1]
        up = np.zeros((px * py, q, q))
        up[:, idx, idx] = part(Nn, j)
        sol = np.linalg.solve(T, np.concatenate([up, rhs], 2))
        U.append(sol[:, :, :q])
        V.append(sol[:, :, q:])
    nxt = None
    for j in range(rows - 1, -1, -1):
        nxt = V[j] if nxt is None else V[j] - U[j] @ nxt
        for k in range(px * py):
            a, b = k % px, k // px
            for comp in range(2):
                out[comp][b * my + 1 + j, a * mx + 1:a * mx + 1 + q] = nxt[k, :, comp]
    return out


def _quality(xi, eta):
    n = xi.shape[0] - 1

    def dx(g):
        return ((g[:-1, 1:] - g[:-1, :-1]) + (g[1:, 1:] - g[1:, :-1])) * 0.5 * n

    def dy(g):
        return ((g[1:, :-1] - g[:-1, :-1]) + (g[1:, 1:] - g[:-1, 1:])) * 0.5 * n

    a, b, c, d = dx(xi), dy(xi), dx(eta), dy(eta)
    skew = np.abs(a * c + b * d) / (np.sqrt(a * a + b * b) * np.sqrt(c * c + d * d))
    return np.array([(a * d - b * c).min(), skew.max()])


def _fit(case, s, seed):
    """The training loop with every product in 64 bits; as in the framework, the network is the weights in BF16."""
    shapes = [(64, 3), (64,), (64, 64), (64,), (64, 64), (64,), (2, 64), (2,)]
    p = torch.from_numpy(_weights(seed)).to(DEV).double()
    m, v, loss = torch.zeros_like(p), torch.zeros_like(p), []
    txy, tgt = s["txy"].double(), s["target"].double()
    j = torch.arange(case["batch"], device=DEV)
    for it in range(1, case["steps"] + 1):
        i = _philox(j, torch.full_like(j, it), torch.zeros_like(j), torch.full_like(j, 2), s["key"])[0] % case["labels"]
        net = p.bfloat16().double().requires_grad_(True)
        w = [q.view(shape) for q, shape in zip(net.split([math.prod(z) for z in shapes]), shapes)]
        z = torch.stack([txy[i, 0] * 20.0 - 1.0, 2.0 * txy[i, 1] - 1.0, 2.0 * txy[i, 2] - 1.0], 1)
        for k in range(0, 6, 2):
            z = torch.tanh(z @ w[k].T + w[k + 1])
        err = ((z @ w[6].T + w[7] - (tgt[i] - txy[i, 1:])) ** 2).mean()
        g, = torch.autograd.grad(err, net)
        m, v = 0.9 * m + 0.1 * g, 0.999 * v + 0.001 * g * g
        p = p - 1e-3 * (m / (1 - 0.9 ** it)) / ((v / (1 - 0.999 ** it)).sqrt() + 1e-8)
        loss.append(err.detach())
    return {"loss": torch.stack(loss), "weights": p}


def exact(case, seed):
    call = case["call"]
    if call in ("batch", "steady", "cv_net"):
        return None   # thousands of steps of every path in turn: minutes
    if call == "train":
        return _fit(case, prepare(case, seed), seed)
    if call == "subdomain":
        s = prepare(case, seed)
        grids = [s[k].cpu().numpy() for k in ("xi", "eta")]
        edges = EQUIDISTRIBUTED if case["edges"] == "equidistributed" else IDENTITY
        return tuple(_subdomains(s["density"], s["t_n"], math.inf if case["steady"] else 5e-4, case["px"], case["py"],
                                 case["cells"], *grids, [v.cpu().numpy() for v in s["iface"]], edges))
    if case["steps"] > 64 or case.get("keys"):
        return None   # a long horizon; a solve at nodes that the step picks itself
    s = prepare(case, seed)
    sim = _simulate(s["density"], s["data"], s["pts"], case["t"], s["dt"], case["paths"], s["key"], 3, s["grids"],
                    case.get("stride", 0))
    if call != "mesh_step":
        return sim
    grids = [s[k].cpu().numpy() for k in ("xi", "eta")]
    new = _subdomains(s["density"], s["t_n"], case["t"], case["px"], case["px"], case["px"] * case["m"], *grids,
                      [sim[k].cpu().numpy() for k in ("xi", "eta")], _edges(case))
    return {"iface_xi": sim["xi"], "iface_eta": sim["eta"], "xi": new[0], "eta": new[1], "quality": _quality(*new)}
