"""Workloads of the library's public entry points, for timing and comparison.

Four kinds of work that programs built on this package do:
  flow   one lattice with red blood cells (Simulation): some coupled steps,
         then a read-out of the cells and, where asked for, of rho and u;
  batch  many independent one-cell boxes in one persistent launch (Batch);
  fit    the shape loss of a batch of boxes and its gradient with respect to
         the membrane stiffnesses and tau (AdjointBoxes, CoupledStepFn);
  pack   force-bias packing of surrogate ellipsoids (Packer).
Sizes are those of the package's own workloads (single cell in shear 32^3,
dense channel 128x64x64, large suspension 256x256x512, 256 calibration boxes
of side 24..48, 64 boxes of 48^3, 10^6 ellipsoids) and ones in between, odd
and ragged sides among them.  All inputs are synthetic and seeded.
"""
import math

import numpy as np
import torch

from paper_2305_02752_amd import Batch, Packer, Simulation
from paper_2305_02752_amd.autograd import AdjointBoxes, CoupledStepFn

K_REF = (1.5e-4, 1.0e-5, 5.0e-2, 1.0e-2)   # link, bend, area, volume stiffness
TRACTION = 4.48e-3                           # 200 pN in lattice units
SEMI = (8.5, 8.5, 3.8)                       # surrogate ellipsoid of a cell
AXES = "xyz"

FLOW = dict(kind="flow", nx=32, ny=32, nz=32, cells=1, steps=10, wall="", wall_u=0.0, body=0.0, le_u=0.0,
            kernel=4, tau=1.0, every=1, ab2=False, ratio=1.0, ratio2=1.0, fields=False)


def listed():
    return [
        # one cell in a sheared box, observed every 20 steps: the smallest program, bound by latency
        dict(FLOW, name="shear_cell_32", steps=20, wall="z", wall_u=0.01, fields=True),
        # body-force channel at dense haematocrit with its fields read out
        dict(FLOW, name="channel_128x64x64", nx=128, ny=64, nz=64, cells=220, steps=200, wall="y", body=1e-5,
             fields=True),
        # the large periodic suspension at 44% haematocrit, cells read out
        dict(FLOW, name="suspension_256x256x512", nx=256, ny=256, nz=512, cells=18600, steps=80, body=1e-6),
        # ragged sides, dilute, forces held over 10 steps and Adams-Bashforth moves
        dict(FLOW, name="ragged_101x75x203_ab2", nx=101, ny=75, nz=203, cells=420, steps=150, body=2e-6, tau=0.9,
             every=10, ab2=True),
        # boundary-free shear with Lees-Edwards images
        dict(FLOW, name="sheared_128x128x128", nx=128, ny=128, nz=128, cells=1160, steps=60, le_u=0.02),
        # channel with healthy and stiffened cells of two interior viscosities
        dict(FLOW, name="stiffened_160x80x80", nx=160, ny=80, nz=80, cells=440, steps=80, wall="z", body=1e-5,
             ratio=5.0, ratio2=10.0),
        # calibration: 256 boxes of side 24..48, one launch per run
        dict(kind="batch", name="calibration_256_boxes", boxes=256, lo=24, hi=48, steps=100, wall="", ratio=1.0,
             tuned=True),
        # a few boxes, sheared between walls, in the default tiling
        dict(kind="batch", name="calibration_6_boxes", boxes=6, lo=24, hi=32, steps=40, wall="z", ratio=5.0,
             tuned=False),
        # parameter fit over 64 boxes, loss and gradient
        dict(kind="fit", name="fit_64x48", boxes=64, side=48, steps=200, ckpt=50),
        # the same for one small box
        dict(kind="fit", name="fit_1x32", boxes=1, side=32, steps=60, ckpt=20),
        # packing of a million ellipsoids
        dict(kind="pack", name="pack_1000000", n=1000000, iters=12, wall="", quad=8, static=False, fraction=0.35),
        # a channel's worth of ellipsoids between walls
        dict(kind="pack", name="pack_6000", n=6000, iters=40, wall="y", quad=8, static=True, fraction=0.3),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(("flow", "flow", "flow", "flow", "batch", "fit", "pack"))
    if kind == "flow":
        form = rng.choice(("periodic", "wall", "sheared"))
        n = [_log(rng, 24, 256) for _ in range(3)]
        if form == "sheared":
            n = [max(24, n[0] // 8 * 8), min(n[1], 160), max(24, n[2] // 8 * 8)]
        if n[0] * n[1] * n[2] > 8_000_000:
            n[rng.randrange(3)] = 32
        sites = n[0] * n[1] * n[2]
        c = dict(FLOW, nx=n[0], ny=n[1], nz=n[2], tau=round(rng.uniform(0.8, 1.2), 3), body=1e-6 * rng.randint(0, 10))
        c["cells"] = max(1, int(sites / 794.0 * rng.uniform(0.05, 0.45)))
        c["steps"] = max(10, min(150, int(2.5e8 / sites)))
        if form == "wall":
            c.update(wall=rng.choice(AXES), wall_u=rng.choice((0.0, 0.01)))
        if form == "sheared":
            c.update(le_u=rng.choice((0.01, 0.02)), body=0.0)
        c["kernel"] = rng.choice((4, 4, 4, 4, 2))
        if rng.random() < 0.25:
            c.update(every=rng.choice((5, 10)), ab2=True)
        if rng.random() < 0.25:
            c["ratio"] = 5.0
            c["ratio2"] = rng.choice((5.0, 10.0))
        c["fields"] = sites < 1_000_000 and rng.random() < 0.5
        return c
    if kind == "batch":
        lo = rng.randint(24, 36)
        return dict(kind="batch", boxes=_log(rng, 4, 200), lo=lo, hi=rng.randint(lo, 48), steps=rng.randint(20, 100),
                    wall=rng.choice(("", "z")), ratio=rng.choice((1.0, 5.0)), tuned=rng.random() < 0.5)
    if kind == "fit":
        boxes = _log(rng, 1, 48)
        ckpt = rng.choice((20, 25, 50))
        return dict(kind="fit", boxes=boxes, side=rng.randint(24, 48), steps=ckpt * rng.randint(2, 3), ckpt=ckpt)
    n = _log(rng, 500, 600_000)
    return dict(kind="pack", n=n, iters=max(5, min(60, 3_000_000 // n)), wall=rng.choice(("", "y", "z")),
                quad=rng.choice((4, 8, 8, 16)), static=n < 150_000, fraction=round(rng.uniform(0.2, 0.4), 2))


# ---------------------------------------------------------------------- inputs
def _mesh():
    """Biconcave cell of diameter 16 (Evans-Fung profile on a level-3
    icosphere): 642 vertices, 1280 triangles, counter-clockwise outside."""
    t = (1.0 + 5.0 ** 0.5) / 2.0
    verts = [(-1, t, 0), (1, t, 0), (-1, -t, 0), (1, -t, 0), (0, -1, t), (0, 1, t), (0, -1, -t), (0, 1, -t),
             (t, 0, -1), (t, 0, 1), (-t, 0, -1), (-t, 0, 1)]
    verts = [np.array(v, dtype=np.float64) / math.sqrt(1.0 + t * t) for v in verts]
    faces = [(0, 11, 5), (0, 5, 1), (0, 1, 7), (0, 7, 10), (0, 10, 11), (1, 5, 9), (5, 11, 4), (11, 10, 2),
             (10, 7, 6), (7, 1, 8), (3, 9, 4), (3, 4, 2), (3, 2, 6), (3, 6, 8), (3, 8, 9), (4, 9, 5), (2, 4, 11),
             (6, 2, 10), (8, 6, 7), (9, 8, 1)]
    for _ in range(3):
        at, out = {}, []

        def mid(a, b):
            key = (min(a, b), max(a, b))
            if key not in at:
                p = verts[a] + verts[b]
                verts.append(p / np.linalg.norm(p))
                at[key] = len(verts) - 1
            return at[key]

        for a, b, c in faces:
            ab, bc, ca = mid(a, b), mid(b, c), mid(c, a)
            out += [(a, ab, ca), (b, bc, ab), (c, ca, bc), (ab, bc, ca)]
        faces = out
    v, tri = np.array(verts), np.array(faces, dtype=np.int32)
    s = v[:, 0] ** 2 + v[:, 1] ** 2
    pos = np.stack([8.0 * v[:, 0], 8.0 * v[:, 1], 4.0 * v[:, 2] * (0.2072 + 2.0026 * s - 1.1228 * s * s)], 1)
    n = np.cross(v[tri[:, 1]] - v[tri[:, 0]], v[tri[:, 2]] - v[tri[:, 0]])   # outward on the sphere
    flip = (n * v[tri].mean(axis=1)).sum(axis=1) < 0
    tri[flip] = tri[flip][:, [0, 2, 1]]
    return pos.astype(np.float32), tri


REST, TRI = _mesh()


class _Lattice:
    """The attributes that Simulation and Batch read from a lattice."""

    def __init__(self, n, wall="", wall_u=0.0, body=0.0, tau=1.0, kernel=4, le_u=0.0):
        self.nx, self.ny, self.nz = (int(v) for v in n)
        self.bc = tuple(1 if a == wall else 0 for a in AXES)
        self.tau, self.ibm_kernel, self.lees_edwards_u = tau, kernel, le_u
        t = (AXES.index(wall) + 1) % 3 if wall else 0    # walls slide, and the flow runs, along a tangential axis
        along = lambda u: tuple(u if d == t else 0.0 for d in range(3))  # noqa: E731
        self.body_force, self.wall_u_lo, self.wall_u_hi = along(body), along(-wall_u), along(wall_u)


def _rotations(n, gen):
    q = torch.randn(n, 4, generator=gen, device="cuda", dtype=torch.float64)
    w, x, y, z = (q / q.norm(dim=1, keepdim=True)).unbind(1)
    return torch.stack([1 - 2 * (y * y + z * z), 2 * (x * y - z * w), 2 * (x * z + y * w),
                        2 * (x * y + z * w), 1 - 2 * (x * x + z * z), 2 * (y * z - x * w),
                        2 * (x * z - y * w), 2 * (y * z + x * w), 1 - 2 * (x * x + y * y)], 1).view(n, 3, 3)


def _place(centres, rots, gen):
    """Cells at the centres: the rest shape stretched by some 5% along its
    own axes (cells in a flow are deformed), turned, with a little vertex
    noise; stiffnesses log-uniform over half a decade."""
    n = centres.shape[0]
    rest = torch.tensor(REST, dtype=torch.float64, device="cuda")
    s = 1.0 + 0.05 * torch.randn(n, 1, 3, generator=gen, device="cuda", dtype=torch.float64).clamp(-2, 2)
    X = torch.einsum("cij,cvj->cvi", rots, rest[None] * s)
    X += 0.02 * torch.randn(X.shape, generator=gen, device="cuda", dtype=torch.float64)
    origin = torch.floor(centres)
    off = (X + (centres - origin)[:, None]).float()
    e = torch.rand(n, 4, generator=gen, device="cuda", dtype=torch.float64) * 0.5 - 0.25
    k = torch.tensor(K_REF, dtype=torch.float64, device="cuda") * 10.0 ** e
    return origin.int().cpu().numpy(), off.cpu().numpy(), k.float().cpu().numpy()


def _grid_centres(case, gen):
    """Jittered grid of centres filling the lattice (off the walls)."""
    n = case["cells"]
    L = np.array([case["nx"], case["ny"], case["nz"]], dtype=np.float64)
    lo = np.array([9.5 if a == case["wall"] else 0.0 for a in AXES])
    hi = np.where(lo > 0, np.maximum(L - 1 - lo, lo), L)
    lo = np.where(lo > 0, np.minimum(lo, 0.5 * (L - 1)), lo)
    hi = np.maximum(hi, lo)
    side = np.maximum(hi - lo, 1.0)
    s = (side.prod() / n) ** (1.0 / 3.0)
    g = np.maximum(1, np.round(side / s)).astype(int)
    while g.prod() < n:
        g[np.argmax(side / g)] += 1
    perm = torch.randperm(int(g.prod()), generator=gen, device="cuda")[:n].cpu().numpy()
    at = np.stack([perm % g[0], perm // g[0] % g[1], perm // (g[0] * g[1])], 1)
    jit = (torch.rand(n, 3, generator=gen, device="cuda", dtype=torch.float64) - 0.5).cpu().numpy()
    c = lo + (at + 0.5 + 0.5 * jit) * (hi - lo) / g
    return torch.tensor(c, dtype=torch.float64, device="cuda")


def _flow_inputs(case, gen):
    lat = _Lattice([case["nx"], case["ny"], case["nz"]], case["wall"], case["wall_u"], case["body"], case["tau"],
                   case["kernel"], case["le_u"])
    cells = _place(_grid_centres(case, gen), _rotations(case["cells"], gen), gen)
    ratio = np.where(np.arange(case["cells"]) % 2 == 0, case["ratio"], case["ratio2"]).astype(np.float32)
    return lat, cells, ratio


def _boxes(sides, wall, tau, gen):
    """One aligned cell near the middle of each cubic box, stretched along x."""
    n = len(sides)
    lats = [_Lattice([s] * 3, wall, 0.01 if wall else 0.0, 0.0, float(t)) for s, t in zip(sides, tau)]
    c = torch.tensor([[(s - 1) / 2.0] * 3 for s in sides], dtype=torch.float64, device="cuda")
    c += torch.rand(n, 3, generator=gen, device="cuda", dtype=torch.float64) - 0.5
    origin, off, k = _place(c, torch.eye(3, dtype=torch.float64, device="cuda").expand(n, 3, 3), gen)
    tr = np.zeros((n, 3), dtype=np.float32)
    tr[:, 0] = TRACTION * torch.rand(n, generator=gen, device="cuda").cpu().numpy()
    return lats, origin, off, k, tr


def _batch_inputs(case, gen):
    span = case["hi"] - case["lo"] + 1
    sides = [case["lo"] + (7 * i) % span for i in range(case["boxes"])]
    return _boxes(sides, case["wall"], [1.0] * case["boxes"], gen)


def _fit_inputs(case, gen):
    b = case["boxes"]
    tau = 0.8 + 0.4 * torch.rand(b, generator=gen, device="cuda", dtype=torch.float64).cpu().numpy()
    inputs = _boxes([case["side"]] * b, "z", tau, gen)
    u = torch.rand(b, 2, generator=gen, device="cuda", dtype=torch.float64).cpu().numpy()
    targets = 16.0 * np.stack([1.0 + 0.5 * u[:, 0], 0.7 + 0.3 * u[:, 1]], 1)
    params = np.concatenate([inputs[3].astype(np.float64), tau[:, None]], 1).astype(np.float32)
    return inputs, targets, params


def _pack_inputs(case, gen):
    n, wall = case["n"], case["wall"]
    side = float(np.float32(max((n * 4.0 / 3.0 * math.pi * math.prod(SEMI) / case["fraction"]) ** (1.0 / 3.0), 40.0)))
    r = (torch.rand(n, 3, generator=gen, device="cuda") * side).contiguous()
    rot = _rotations(n, gen).float().contiguous()
    semi = torch.tensor(SEMI, device="cuda") * (1.0 - 0.15 * torch.rand(n, 1, generator=gen, device="cuda"))
    dom = dict(box=(side,) * 3, periodic=tuple(a != wall for a in AXES), lo=(0.0,) * 3, hi=(side,) * 3, max_semi=9.0,
               eta=0.03, max_move=1.0, quad=case["quad"])
    return r, rot, semi.contiguous(), dom


class _Cells:
    def __init__(self, origin, offsets, k, traction):
        self.origin, self.offsets, self.k, self.traction = origin, offsets, k, traction


def prepare(case, seed):
    gen = torch.Generator(device="cuda").manual_seed(seed)
    if case["kind"] == "flow":
        lat, (origin, off, k), ratio = _flow_inputs(case, gen)
        sim = Simulation(lat, REST, TRI, max_cells=case["cells"])
        sim.set_cells(origin, off, k)
        sim.set_integration(case["every"], "ab2" if case["ab2"] else "euler")
        sim.set_field_output(case["fields"])
        if case["ratio"] != case["ratio2"]:
            sim.set_cell_viscosity(ratio)
        elif case["ratio"] != 1.0:
            sim.set_interior_viscosity(case["ratio"])
        return case, sim
    if case["kind"] == "batch":
        lats, origin, off, k, tr = _batch_inputs(case, gen)
        batch = Batch(lats, REST, TRI)
        batch.set_cells(origin, off, k, tr)
        if case["ratio"] != 1.0:
            batch.set_interior_viscosity(case["ratio"])
        if case["tuned"]:   # as a program does that runs one batch shape many times
            batch.autotune(trial_steps=10)
        return case, batch
    if case["kind"] == "fit":
        (lats, origin, off, k, tr), targets, params = _fit_inputs(case, gen)
        cells = [_Cells(origin[b:b + 1], off[b:b + 1], k[b:b + 1], tr[b:b + 1]) for b in range(case["boxes"])]
        return case, AdjointBoxes(lats, REST, TRI, cells, targets, case["steps"], case["ckpt"]), torch.tensor(params)
    r, rot, semi, dom = _pack_inputs(case, gen)
    return case, Packer(**dom), r, rot, semi


def run(state):
    case = state[0]
    if case["kind"] == "flow":
        sim = state[1]
        sim.step(case["steps"])
        origin, off, force = sim.read_vertices()
        out = {"origin": origin, "offsets": off, "force": force, "velocity": sim.read_vertex_velocity()}
        if case["fields"]:
            out["rho"], out["u"] = sim.read_macro()
        return out
    if case["kind"] == "batch":
        batch = state[1]
        batch.run(case["steps"])
        batch.sync()
        cells = [batch.read_vertices(b) for b in range(case["boxes"])]
        return {n: np.stack([c[i] for c in cells]) for i, n in ((1, "offsets"), (2, "force"), (3, "velocity"))}
    if case["kind"] == "fit":
        params = state[2].clone().requires_grad_(True)
        loss = CoupledStepFn.apply(params, state[1])
        loss.sum().backward()
        return {"loss": loss.detach(), "grad": params.grad}
    packer, r, rot, semi = state[1:]
    centres = r.clone()
    go = packer.run_device_static if case["static"] else packer.run_device
    overlap = go(centres, rot, semi, case["iters"])
    return {"centres": centres, "pairs": [int(overlap[1]), int(overlap[3])],
            "volume": np.array([overlap[0], overlap[2]], dtype=np.float32)}


def work(case):
    if case["kind"] == "pack":
        # centres in and out, orientations and semi-axes in; some 3 close pairs an ellipsoid, both ways over the points
        points = {4: 32, 8: 280, 16: 2176}[case["quad"]]
        return {"bytes": 72.0 * case["n"] * case["iters"], "flops": 3.0 * 2 * 24 * points * case["n"] * case["iters"]}
    if case["kind"] == "flow":
        sites, cells = case["nx"] * case["ny"] * case["nz"], case["cells"]
    elif case["kind"] == "batch":
        span = case["hi"] - case["lo"] + 1
        sites, cells = sum((case["lo"] + (7 * i) % span) ** 3 for i in range(case["boxes"])), case["boxes"]
    else:
        sites, cells = case["boxes"] * case["side"] ** 3, case["boxes"]
    # 19 populations in and out a site and step, positions in and out a vertex; some 250 operations a site
    # (moments, equilibrium, forcing) and 64 x 14 + 750 a vertex (both IBM directions, three hinges)
    step = {"bytes": 152.0 * sites + 24.0 * 642 * cells, "flops": 250.0 * sites + 1650.0 * 642 * cells}
    if case["kind"] == "fit":
        # forward, recomputation, and the collision's transpose (19 cotangents in and out, populations, force in)
        step = {"bytes": 2 * step["bytes"] + 264.0 * sites, "flops": 4 * step["flops"]}
    return {k: v * case["steps"] for k, v in step.items()}


# ---------------------------------------------------------------------- 64-bit values
_C = np.array([[0, 0, 0], [1, 0, 0], [-1, 0, 0], [0, 1, 0], [0, -1, 0], [0, 0, 1], [0, 0, -1], [1, 1, 0], [-1, -1, 0],
               [1, -1, 0], [-1, 1, 0], [1, 0, 1], [-1, 0, -1], [1, 0, -1], [-1, 0, 1], [0, 1, 1], [0, -1, -1],
               [0, 1, -1], [0, -1, 1]])
_OPP = [0] + [i + 1 if i % 2 else i - 1 for i in range(1, 19)]


def _topology():
    wing = {}
    for a, b, c in TRI.tolist():
        wing[(a, b)], wing[(b, c)], wing[(c, a)] = c, a, b
    return torch.tensor([(p, q, wing[(p, q)], wing[(q, p)]) for p, q in sorted(wing) if p < q], device="cuda").T


class _Model:
    """The coupled step in float64: membrane forces, spreading, BGK with
    Guo's forcing, interpolation, move.  X [C, V, 3] absolute positions,
    g [19, nz, ny, nx] populations less their weights, before a collision."""

    def __init__(self, lat, origin, off, k, traction=None, ratio=None):
        f64 = lambda v: torch.tensor(np.asarray(v, dtype=np.float32), dtype=torch.float64, device="cuda")  # noqa: E731
        self.lat, self.n = lat, (lat.nx, lat.ny, lat.nz)
        self.X = f64(off) + torch.tensor(origin, dtype=torch.float64, device="cuda")[:, None]
        self.k, self.tau, self.traction = f64(k), f64(lat.tau), None if traction is None else f64(traction)
        self.ratio = None if ratio is None or np.all(ratio == 1.0) else f64(ratio)
        self.c = torch.tensor(_C, dtype=torch.float64, device="cuda")
        self.w = f64([0.0] * 19) + torch.tensor([1 / 3] + [1 / 18] * 6 + [1 / 36] * 12, dtype=torch.float64, device="cuda")
        self.body, self.wall = f64(lat.body_force), (f64(lat.wall_u_lo), f64(lat.wall_u_hi))
        self.tri, self.hinge = torch.tensor(TRI, device="cuda").long().T, _topology()
        rest = f64(REST)[None]
        self.L0, self.th0 = self.edges(rest), self.angles(rest)
        self.A0, self.V0 = self.area_volume(rest)
        idx = np.arange(len(REST))
        x = REST.astype(np.float64)[:, 0]
        self.pole = torch.zeros(len(REST), dtype=torch.float64, device="cuda")
        self.pole[np.lexsort((idx, -x))[:32]], self.pole[np.lexsort((idx, x))[:32]] = 1 / 32, -1 / 32

    def edges(self, X):
        return (X[:, self.hinge[1]] - X[:, self.hinge[0]]).norm(dim=-1)

    def angles(self, X):
        xi, xj, xk, xl = (X[:, h] for h in self.hinge)
        n1 = torch.cross(xj - xi, xk - xi, dim=-1)
        n2 = torch.cross(xi - xj, xl - xj, dim=-1)
        e = (xj - xi) / (xj - xi).norm(dim=-1, keepdim=True)
        return torch.atan2((torch.cross(n1, n2, dim=-1) * e).sum(-1), (n1 * n2).sum(-1))

    def area_volume(self, X):
        a, b, c = (X[:, t] - X[:, :1].detach() for t in self.tri)
        return (0.5 * torch.cross(b - a, c - a, dim=-1).norm(dim=-1).sum(-1),
                (a * torch.cross(b, c, dim=-1)).sum(-1).sum(-1) / 6.0)

    def forces(self, X):
        """Minus the gradient of the membrane energy (inside its clamps), with the pole traction."""
        graph = torch.is_grad_enabled() and (X.requires_grad or self.k.requires_grad)
        with torch.enable_grad():
            Y = X if X.requires_grad else X.detach().requires_grad_(True)
            s, d = (self.edges(Y) - self.L0) / self.L0, self.angles(Y) - self.th0
            (A, V), k, tb = self.area_volume(Y), self.k, math.pi / 6
            E = (k[:, 0] * (self.L0 * (0.5 * s * s - 0.5 * torch.log(1 - s * s / 9))).sum(-1)
                 + k[:, 1] * (0.5 * d * d - 0.5 * torch.log(1 - d * d / tb ** 2)).sum(-1)
                 + 0.5 * k[:, 2] * self.A0 * ((A - self.A0) / self.A0) ** 2
                 + 0.5 * k[:, 3] * self.V0 * ((V - self.V0) / self.V0) ** 2).sum()
            F = -torch.autograd.grad(E, Y, create_graph=graph)[0]
        F = F if graph else F.detach()
        return F if self.traction is None else F + self.pole[:, None] * self.traction[:, None]

    def stencil(self, X, delta):
        """Sites [M, K^3], weights (zero past a wall), the wall's share, and the image of each node."""
        K, lat = self.lat.ibm_kernel, self.lat
        at = torch.arange(-1, 3, device="cuda") if K == 4 else torch.arange(0, 2, device="cuda")

        def axis(x):
            node = torch.floor(x.detach()).long()[..., None] + at
            r = (x[..., None] - node).abs()
            if K == 2:
                return node, 1 - r
            q = torch.where(r < 1, 1 + 4 * r - 4 * r * r, -7 + 12 * r - 4 * r * r).clamp_min(1e-30).sqrt()
            return node, torch.where(r < 1, (3 - 2 * r + q) / 8, (5 - 2 * r - q) / 8)

        (iy, wy), (iz, wz) = axis(X[:, 1]), axis(X[:, 2])
        image = torch.div(iz, lat.nz, rounding_mode="floor") if lat.lees_edwards_u else torch.zeros_like(iz)
        ix, wx = axis(X[:, None, 0] - image * delta)             # [M, K (z), K (x)]
        idx = [ix[:, :, None, :], iy[:, None, :, None], iz[:, :, None, None]]
        W = wz[:, :, None, None] * wy[:, None, :, None] * wx[:, :, None, :]
        side, site = 0, 0
        for d in (2, 1, 0):
            if lat.bc[d]:
                side = (idx[d] < 0).long() + 2 * (idx[d] >= self.n[d]).long() + torch.zeros_like(W, dtype=torch.long)
                p = idx[d].clamp(0, self.n[d] - 1)
            else:
                p = idx[d] % self.n[d]
            site = site * self.n[d] + p
        M = X.shape[0]
        flat = lambda v: (v + torch.zeros_like(W, dtype=v.dtype)).reshape(M, -1)  # noqa: E731
        wall = [(W * (side == s)).reshape(M, -1).sum(1) if any(lat.bc) else None for s in (1, 2)]
        W = W * (side == 0) if any(lat.bc) else W
        return flat(site), W.reshape(M, -1), wall, flat(image[:, :, None, None])

    def inside(self, X, delta):
        """Largest viscosity ratio of the cells holding each site (1 outside), by parity along z."""
        lat, C = self.lat, X.shape[0]
        lo = torch.floor(X.amin(1)).long() - 1
        n = (torch.floor(X.amax(1)).long() + 3 - lo).amax(0).tolist()
        t = (X - lo[:, None])[:, self.tri.T]                          # [C, T, 3, 3]
        base = torch.floor(t[..., :2].amin(2)).long()
        reach = int((torch.floor(t[..., :2].amax(2)).long() - base).max()) + 1
        flips = torch.zeros(C * n[0] * n[1] * n[2], dtype=torch.int32, device="cuda")
        for px in range(reach + 1):
            for py in range(reach + 1):
                p = base + torch.tensor([px, py], device="cuda")
                q = t[..., :2] - p[:, :, None].double()
                s = [q[..., a, 0] * q[..., b, 1] - q[..., a, 1] * q[..., b, 0] for a, b in ((1, 2), (2, 0), (0, 1))]
                area = s[0] + s[1] + s[2]
                hit = ((s[0] > 0) & (s[1] > 0) & (s[2] > 0)) | ((s[0] < 0) & (s[1] < 0) & (s[2] < 0))
                z = sum(s[a] * t[..., a, 2] for a in range(3)) / torch.where(hit, area, torch.ones_like(area))
                c, k = hit.nonzero(as_tuple=True)
                at = ((c * n[1] + p[c, k, 1]) * n[0] + p[c, k, 0]) * n[2] + torch.ceil(z[c, k]).long()
                flips.index_add_(0, at, torch.ones_like(at, dtype=torch.int32))
        odd = (flips.view(C, n[1], n[0], n[2]).cumsum(3) % 2).nonzero()
        c, node = odd[:, 0], [odd[:, 2] + lo[odd[:, 0], 0], odd[:, 1] + lo[odd[:, 0], 1], odd[:, 3] + lo[odd[:, 0], 2]]
        keep = torch.ones_like(c, dtype=torch.bool)
        site = 0
        for d in (2, 1, 0):
            if lat.bc[d]:
                keep &= (node[d] >= 0) & (node[d] < self.n[d])
            site = site * self.n[d] + node[d] % self.n[d]
        out = torch.ones(lat.nx * lat.ny * lat.nz, dtype=torch.float64, device="cuda")
        return out.scatter_reduce(0, site[keep], self.ratio[c[keep]], "amax").view(lat.nz, lat.ny, lat.nx)

    def stream(self, h, rho, delta):
        lat, out = self.lat, []
        for q in range(19):
            o = torch.roll(h[q], tuple(int(v) for v in _C[q][::-1]), (0, 1, 2))
            d = lat.bc.index(1) if any(lat.bc) else 2
            e = int(_C[q][d])
            if e and any(lat.bc):
                at = [slice(None)] * 3
                at[2 - d] = 0 if e > 0 else self.n[d] - 1
                j = _OPP[q]
                o = o.clone()
                o[tuple(at)] = h[j][tuple(at)] - 6 * self.w[j] * rho[tuple(at)] * (self.c[j] @ self.wall[0 if e > 0 else 1])
            elif e and lat.lees_edwards_u:
                to, src, sign = (0, lat.nz - 1, -1.0) if e > 0 else (lat.nz - 1, 0, 1.0)
                pos = torch.arange(lat.nx, device="cuda").double() - int(_C[q][0]) - sign * delta
                x0 = torch.floor(pos)
                s, x0 = pos - x0, x0.long() % lat.nx
                row = torch.roll(h[:, src], int(_C[q][1]), 1)
                g = (1 - s) * row[:, :, x0] + s * row[:, :, (x0 + 1) % lat.nx]
                r = 1 + g.sum(0)
                u = torch.tensordot(self.c.T, g, 1) / r
                v = u.clone()
                v[0] += sign * lat.lees_edwards_u
                o = o.clone()
                o[to] = g[q] + self.feq(r, v)[q] - self.feq(r, u)[q]
            out.append(o)
        return torch.stack(out)

    def feq(self, rho, u):
        sh = (19,) + (1,) * rho.dim()
        eu = torch.tensordot(self.c, u, 1)
        return self.w.view(sh) * ((rho - 1) + rho * (3 * eu + 4.5 * eu * eu - 1.5 * (u * u).sum(0)))

    def run(self, steps, every=1, ab2=False):
        lat, X = self.lat, self.X
        C, N = X.shape[0], lat.nx * lat.ny * lat.nz
        g = torch.zeros(19, lat.nz, lat.ny, lat.nx, dtype=torch.float64, device="cuda")
        U = prev = None
        for t in range(steps):
            delta = (lat.lees_edwards_u * t) % lat.nx
            Fv = self.forces(X) if t % every == 0 else Fv
            site, W, wall, image = self.stencil(X.reshape(-1, 3), delta)
            F = torch.zeros(N, 3, dtype=torch.float64, device="cuda").index_add(
                0, site.reshape(-1), (W[:, :, None] * Fv.reshape(-1, 1, 3)).reshape(-1, 3))
            F = (F + self.body).T.view(3, lat.nz, lat.ny, lat.nx)
            rho = 1 + g.sum(0)
            u = (torch.tensordot(self.c.T, g, 1) + 0.5 * F) / rho
            uv = u.reshape(3, N).T[site]
            if lat.lees_edwards_u:
                uv = uv + torch.stack([image * lat.lees_edwards_u, 0 * image, 0 * image], 2)
            prev, U = U, (W[:, :, None] * uv).sum(1)
            if any(lat.bc):
                U = U + wall[0][:, None] * self.wall[0] + wall[1][:, None] * self.wall[1]
            U = U.view(X.shape)
            om = 1 / (self.tau if self.ratio is None else 0.5 + self.inside(X, delta) * (self.tau - 0.5))
            eu, eF = torch.tensordot(self.c, u, 1), torch.tensordot(self.c, F, 1)
            S = self.w.view(19, 1, 1, 1) * (3 * eF - 3 * (u * F).sum(0) + 9 * eu * eF)
            g = self.stream(g - om * (g - self.feq(rho, u)) + (1 - 0.5 * om) * S, rho, delta)
            X = X + (1.5 * U - 0.5 * prev if ab2 and prev is not None else U)
        return X, Fv, U, rho, u


def exact(case, seed):
    gen = torch.Generator(device="cuda").manual_seed(seed)
    if case["kind"] == "flow":
        # too long beyond; the marking of sheared images is not repeated here
        if case["nx"] * case["ny"] * case["nz"] * case["steps"] > 4e8 or (case["le_u"] and case["ratio"] != 1.0):
            return None
        lat, (origin, off, k), ratio = _flow_inputs(case, gen)
        with torch.no_grad():
            X, Fv, U, rho, u = _Model(lat, origin, off, k, ratio=ratio).run(case["steps"], case["every"], case["ab2"])
            out = {"origin": None, "offsets": X - torch.tensor(origin, device="cuda")[:, None], "force": Fv, "velocity": U}
        return dict(out, rho=rho, u=u) if case["fields"] else out
    if case["kind"] == "batch":
        if case["boxes"] * case["steps"] > 400:
            return None
        lats, origin, off, k, tr = _batch_inputs(case, gen)
        got = []
        with torch.no_grad():
            for b, lat in enumerate(lats):
                one = slice(b, b + 1)
                X, Fv, U, _, _ = _Model(lat, origin[one], off[one], k[one], tr[one],
                                        np.array([case["ratio"]], dtype=np.float32)).run(case["steps"])
                got.append((X - torch.tensor(origin[one], device="cuda")[:, None], Fv, U))
        return {n: torch.cat([v[i] for v in got]) for i, n in enumerate(("offsets", "force", "velocity"))}
    if case["kind"] == "fit":
        if case["boxes"] * case["steps"] * case["side"] ** 3 > 1e7:
            return None
        (lats, origin, off, k, tr), targets, params = _fit_inputs(case, gen)
        losses, grads = [], []
        for b, lat in enumerate(lats):
            one = slice(b, b + 1)
            m = _Model(lat, origin[one], off[one], k[one], tr[one])
            p = torch.tensor(params[b].astype(np.float64), device="cuda", requires_grad=True)
            m.k, m.tau = p[None, :4], p[4]
            X = m.run(case["steps"])[0][0]
            ext = [X[:, d].max() - X[:, d].min() - targets[b, d] for d in (0, 1)]
            loss = ext[0] ** 2 + ext[1] ** 2
            loss.backward()
            losses.append(loss.detach())
            grads.append(p.grad)
        return {"loss": torch.stack(losses), "grad": torch.stack(grads)}
    if case["n"] > 20000:
        return None   # every pair is looked at below
    r, rot, semi, dom = _pack_inputs(case, gen)
    r, R, s = r.double(), rot.double(), semi.double()
    L, per = dom["box"][0], torch.tensor(dom["periodic"], device="cuda")
    m = case["quad"]
    a = (2 * torch.arange(m, device="cuda").double() + 1) / m - 1
    pts = torch.cartesian_prod(a, a, a)
    pts = pts[(pts * pts).sum(1) <= 1]
    vol = 4.0 / 3.0 * math.pi * s.prod(1)
    ext = (R * R * (s * s)[:, None, :]).sum(2).sqrt()
    near = s.amax(1)

    def overlaps(r):
        i, j = [], []
        for at in range(0, case["n"], 2000):
            d = r[at:at + 2000, None] - r[None]
            d = torch.where(per, d - L * torch.round(d / L), d)
            p, q = ((d * d).sum(2) < (near[at:at + 2000, None] + near) ** 2).nonzero(as_tuple=True)
            keep = p + at < q
            i.append(p[keep] + at)
            j.append(q[keep])
        i, j = torch.cat(i), torch.cat(j)
        d = r[i] - r[j]
        d = torch.where(per, d - L * torch.round(d / L), d)
        V = []
        for at in range(0, len(i), 50000):
            e = slice(at, at + 50000)
            n = []
            for p, q, dd in ((i[e], j[e], d[e]), (j[e], i[e], -d[e])):
                x = torch.einsum("cij,ckj->cki", R[p], pts[None] * s[p][:, None]) + dd[:, None]
                y = torch.einsum("cij,cki->ckj", R[q], x) / s[q][:, None]
                n.append(((y * y).sum(2) <= 1).sum(1).double())
            V.append((vol[i[e]] * n[0] + vol[j[e]] * n[1]) / (2 * len(pts)))
        return i, j, d, torch.cat(V)

    total = []
    for it in range(case["iters"] + 1):
        i, j, d, V = overlaps(r)
        if it in (0, case["iters"]):
            total.append(V.sum())
        if it == case["iters"]:
            break
        f = (dom["eta"] * V / d.norm(dim=1).clamp_min(1e-300))[:, None] * d
        move = torch.zeros_like(r).index_add(0, i, f).index_add(0, j, -f)
        n = move.norm(dim=1, keepdim=True)
        r = r + move * (dom["max_move"] / n.clamp_min(1e-300)).clamp_max(1.0)
        r = torch.where(per, r % L, torch.minimum(torch.maximum(r, ext), L - ext))
    return {"centres": r, "pairs": [None, None], "volume": torch.stack(total)}
