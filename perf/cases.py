"""Timed workloads of the framework's public calls.

Each case is one pass through the entry points a program uses: a time step of
an adaptively refined hierarchy (1D, 2D, 3D; primitive WENO5), the right-hand
side alone (characteristic WENO5), the gradient tagger, a regrid, the
velocity-gradient output, and the refinement predictor's training step and
inference.  The meshes follow the fronts of the initial data: balls (intervals
in 1D, discs in 2D) whose surfaces are refined to the finest level, as the
tagger refines a blast front.

``exact`` evaluates the same passes from the definitions of the method in
plain torch float64 on the CPU, sharing no code with the package.
"""
import itertools
import math
import random

import numpy as np
import torch

GAMMA, CFL, EPS, THETA, BUFFER, NG = 1.4, 0.5, 1e-6, 0.02, 2, 4
F64 = torch.float64


# ---------------------------------------------------------------------------
# the cases
# ---------------------------------------------------------------------------
def _mesh_case(kind, dim, base, patches, balls, radius, **kw):
    """``base`` level-0 cells per dimension, ``patches`` the patch edge of each
    level, ``balls`` fronts of about ``radius`` at places that ``places`` gives."""
    return dict(kind=kind, dim=dim, base=base, patches=patches, balls=balls, radius=radius, places=0,
                periodic=True, scheme="weno", graph=False) | kw


def listed():
    return [
        # the 1D shock-tube run: a few hundred cells, launches and latency
        dict(name="step_1d", **_mesh_case("step", 1, 256, "16,16", 1, 0.15, periodic=False)),
        # the 2D three-level run (256^2 base, 32/16/16 patches), steps replayed as a graph
        dict(name="step_2d", **_mesh_case("step", 2, 256, "32,16,16", 4, 0.12, graph=True)),
        # the 2D five-level run (512^2 base, 32^2 patches), eager steps between regrids
        dict(name="step_2d_deep", **_mesh_case("step", 2, 512, "32,32,32,32,32", 3, 0.08)),
        # a small 3D hierarchy, as the accuracy runs and a regrid's first steps have it
        dict(name="step_3d_small", **_mesh_case("step", 3, 32, "16,16,8", 1, 0.12)),
        # the 3D four-level layout of the headline benchmark (32/16/16/8 patches), millions of cells
        dict(name="step_3d_large", **_mesh_case("step", 3, 64, "32,16,16,8", 8, 0.08)),
        # the shock-capturing scheme's right-hand side; an edge that only the smallest tile divides
        dict(name="rhs_3d_char", **_mesh_case("rhs", 3, 48, "12,12", 2, 0.15, scheme="char")),
        # the tagger as judge after every step of a learned regridding policy
        dict(name="tag_3d", **_mesh_case("tag", 3, 64, "32,16,16,8", 4, 0.08, cells=False)),
        # refinement and coarsening of a front that moves
        dict(name="regrid_3d", **_mesh_case("regrid", 3, 64, "16,16,8", 3, 0.12)),
        # flow output (velocity gradient, numerical schlieren) between transmissive walls, ragged patches
        dict(name="gradient_2d", **_mesh_case("gradient", 2, 240, "24,24,24", 3, 0.12, periodic=False)),
        # one training batch of the predictor
        dict(name="train_2d", kind="train", dim=2, edge=16, tiles=64),
        dict(name="train_3d", kind="train", dim=3, edge=8, tiles=64),
        # the predictor over the finest patches of a hierarchy: input tiles and logits
        dict(name="predict_3d", **_mesh_case("predict", 3, 64, "16,16,8", 2, 0.12, tiles=256)),
    ]


def _log(rng, lo, hi):
    return math.exp(rng.uniform(math.log(lo), math.log(hi)))


def draw(rng):
    kind = rng.choice(["step", "step", "step", "rhs", "tag", "regrid", "gradient", "train", "predict"])
    if kind == "train":
        dim = rng.choice([2, 3])
        return dict(kind=kind, dim=dim, edge=rng.choice([8, 12, 16, 22, 32]) if dim == 2 else 8,
                    tiles=int(_log(rng, 1, 257)))
    dim = rng.choice([2, 3]) if kind == "predict" else rng.choice([1, 2, 2, 3, 3, 3])
    layouts = {1: ["16,16", "8,8,8", "24,16", "40"], 2: ["32,16,16", "16,16", "24,24,24", "32,32,32", "8,16"],
               3: ["16,16,8", "32,16,16,8", "12,12", "8,8,8", "16", "24,16"]}[dim]
    if kind == "regrid":
        layouts = [p for p in layouts if "," in p]
    if kind == "predict":
        layouts = [p for p in layouts if p.split(",")[-1] == ("16" if dim == 2 else "8") and "," in p]
    patches = rng.choice(layouts)
    n = [int(v) for v in patches.split(",")]
    unit = math.lcm(*[v if l == 0 else max(1, v // math.gcd(v, 2 ** l)) for l, v in enumerate(n)])
    lo, hi = {1: (64, 8192), 2: (64, 400), 3: (24, 64 if len(n) > 1 else 160)}[dim]
    base = unit * max(2, round(_log(rng, lo, hi) / unit))
    if dim == 3 and len(n) > 3:
        base = 64
    if kind == "regrid" and len(n) < 4:
        base = max(base, unit * -(-4 * n[0] // unit))
    kw = dict(periodic=rng.random() < 0.7)
    if kind in ("step", "rhs"):
        kw["scheme"] = rng.choice(["weno", "weno", "weno", "char", "central"])
    if kind == "step":
        kw["graph"] = rng.random() < 0.4
    if kind == "tag":
        kw["cells"] = len(n) < 3 or rng.random() < 0.5
    if kind == "predict":
        kw["tiles"] = int(_log(rng, 1, 256))
    balls = 1 if dim == 1 or kind == "regrid" else rng.randint(1, 4)
    return _mesh_case(kind, dim, base, patches, balls, round(rng.uniform(0.08, 0.13), 4), places=rng.randrange(1, 10**6), **kw)


# ---------------------------------------------------------------------------
# the mesh of a case: which patches exist, in the order the library creates them
# ---------------------------------------------------------------------------
def _fronts(case):
    """Centre and radius of each ball."""
    rng = random.Random(1000 + case["places"])
    return [([rng.uniform(0.25, 0.75) if case["dim"] == 1 else rng.random() for _ in range(case["dim"])],
             case["radius"] * rng.uniform(0.95, 1.05)) for _ in range(case["balls"])]


class Mesh:
    """Patches by level.  ``coords[l]``: positions (x, y, z) in creation order,
    which is the order of their slots in the level's pool."""

    def __init__(self, case):
        self.dim, self.periodic = case["dim"], case["periodic"]
        self.n = [int(v) for v in case["patches"].split(",")]
        self.nlev = len(self.n)
        self.cells = [case["base"] << l for l in range(self.nlev)]
        self.np = [c // n for c, n in zip(self.cells, self.n)]
        self.coords = [[] for _ in self.n]
        self.index = [{} for _ in self.n]
        self.parents = [set() for _ in self.n]   # patches with children
        self.rounds = []                         # (level, positions) of each refinement round
        for c in itertools.product(range(self.np[0]), repeat=self.dim):
            self._add(0, tuple(reversed(c)))
        self.moore = [tuple(reversed(o)) for o in itertools.product((-1, 0, 1), repeat=self.dim) if any(o)]
        for l in range(self.nlev - 1):
            want = self._near(l, _fronts(case))
            self.rounds.append((l, want))
            for c in want:
                self.refine(l, c)

    def _add(self, l, c):
        self.index[l][c] = len(self.coords[l])
        self.coords[l].append(c)

    def neighbour(self, l, c, o):
        q = [a + b for a, b in zip(c, o)]
        if self.periodic:
            return tuple(v % self.np[l] for v in q)
        return tuple(q) if all(0 <= v < self.np[l] for v in q) else None

    def refine(self, l, c):
        """A patch is refined once its neighbours on its own level all exist."""
        if c in self.parents[l]:
            return
        for o in self.moore:
            q = self.neighbour(l, c, o)
            if q is not None and q not in self.index[l]:
                self.refine(l - 1, tuple(v * self.n[l] // 2 // self.n[l - 1] for v in q))
        r = 2 * self.n[l] // self.n[l + 1]
        self.parents[l].add(c)
        for o in itertools.product(range(r), repeat=self.dim):
            self._add(l + 1, tuple(a * r + b for a, b in zip(c, reversed(o))))

    def _near(self, l, fronts):
        """Patches of level l that a front crosses, by (z, y, x)."""
        a = np.array(self.coords[l]).reshape(-1, self.dim)
        x = (a + 0.5) * self.n[l] / self.cells[l]
        reach = (0.5 * self.n[l] + 2) / self.cells[l] * math.sqrt(self.dim)
        hit = np.zeros(len(a), bool)
        for c, r in fronts:
            d = x - np.array(c)
            if self.periodic:
                d -= np.round(d)
            hit |= np.abs(np.sqrt((d * d).sum(1)) - r) <= reach
        return sorted((tuple(int(v) for v in c) for c in a[hit]), key=lambda c: c[::-1])

    def complete(self, l):
        """Leaves of level l whose neighbours all exist, by (z, y, x)."""
        ok = [c for c in self.coords[l] if c not in self.parents[l]
              and all(q is None or q in self.index[l] for q in (self.neighbour(l, c, o) for o in self.moore))]
        return sorted(ok, key=lambda c: c[::-1])

    def leaf_cells(self):
        return sum((len(c) - len(p)) * n ** self.dim for c, p, n in zip(self.coords, self.parents, self.n))

    def all_cells(self):
        return sum(len(c) * n ** self.dim for c, n in zip(self.coords, self.n))

    def leaves(self, l):
        return torch.tensor([c not in self.parents[l] for c in self.coords[l]])

    def extra(self):
        """Patches a regrid pass adds: one in four of the leaves it may refine."""
        if self.nlev < 2:
            return []
        for l in range(self.nlev - 2, -1, -1):
            if (ok := self.complete(l)):
                return [(l, c) for c in ok[::4]]
        return []


def _primitives(case, seed, mesh, l, device):
    """Density, velocity components and pressure at the cell centres of the
    level's patches: [P, n, ...] in (z, y, x) order."""
    d, n = mesh.dim, mesh.n[l]
    co = torch.tensor(mesh.coords[l], dtype=torch.int64).reshape(-1, d).to(device)
    x = []
    for j in range(d):
        g = co[:, j:j + 1] * n + torch.arange(n, device=device)
        shape = [len(mesh.coords[l])] + [1] * d
        shape[d - j] = n
        x.append(((g.to(F64) + 0.5) / mesh.cells[l]).reshape(shape))
    full = [len(mesh.coords[l])] + [n] * d
    rng = random.Random(2000 + seed)
    field = []
    for _ in range(1 + d):   # a few long waves each for the density and the velocities
        f = torch.zeros(full, dtype=F64, device=device)
        for _ in range(4):
            k = [rng.randint(-3, 3) for _ in range(d)]
            ph = sum((2 * math.pi * k[j]) * x[j] for j in range(d)) + rng.uniform(0, 2 * math.pi)
            f += torch.cos(ph) * rng.uniform(0.0, 0.05)
        field.append(f)
    rho, p = 1.0 + field[0], torch.ones(full, dtype=F64, device=device)
    for c, r in _fronts(case):
        rj, pj = rng.uniform(0.5, 1.5), (rng.uniform(5.0, 20.0) if d == 3 else rng.uniform(0.2, 1.5))
        # the front has moved a little since the mesh was made
        moved = [rng.uniform(-0.02, 0.02) for _ in range(d)]
        r2 = 0
        for j in range(d):
            dx = x[j] - c[j] - moved[j]
            r2 = r2 + ((dx - torch.round(dx)) if mesh.periodic else dx) ** 2
        inside = r2 < r * r
        rho = torch.where(inside, rj * rho, rho)
        p = torch.where(inside, torch.full_like(p, pj), p)
    return rho, field[1:], p


def _conserved(rho, u, p):
    ke = sum(v * v for v in u)
    return torch.stack([rho] + [rho * v for v in u] + [p / (GAMMA - 1.0) + 0.5 * rho * ke], 1)


# ---------------------------------------------------------------------------
# what a program holds, and one pass
# ---------------------------------------------------------------------------
def _hierarchy(case, seed):
    from paper_2508_05020_amd import amr, workloads

    mesh = Mesh(case)
    extra = mesh.extra() if case["kind"] == "regrid" else []
    cap = [len(c) for c in mesh.coords]
    for l, _ in extra:
        cap[l + 1] += (2 * mesh.n[l] // mesh.n[l + 1]) ** mesh.dim
    # slots for every patch and for the refinement that a run has in reserve
    cap = [c if l == 0 else c + 64 + c // 8 for l, c in enumerate(cap)]
    cfg = workloads.AMRConfig(name="case", dim=mesh.dim, base_cells=case["base"], patch_cells=mesh.n,
                              periodic=[mesh.periodic] * mesh.dim, gamma=GAMMA, cfl=CFL, weno_eps=EPS, tag_theta=THETA,
                              tag_buffer=BUFFER, max_patches=sum(cap), level_capacity=tuple(cap))
    scheme = {"weno": amr.SCHEME_WENO, "char": amr.SCHEME_CHAR, "central": amr.SCHEME_CENTRAL}[case["scheme"]]
    h = amr.Hierarchy(cfg, scheme=scheme)
    # slots are dealt per level: the capacity is at most the level's patches
    cap = [min(c, p ** mesh.dim) for c, p in zip(cap, mesh.np)]
    first = [sum(cap[:l]) for l in range(mesh.nlev)]
    none = np.zeros(cfg.max_patches, np.uint8)
    for l, want in mesh.rounds:
        flags = none.copy()
        flags[[first[l] + mesh.index[l][c] for c in want]] = 1
        h.regrid(flags, none)
    if h.counts()[0] != sum(len(c) for c in mesh.coords):
        raise RuntimeError("the hierarchy is not the case's mesh")
    u = h.state_tensor(0)
    for l in range(mesh.nlev):
        if mesh.coords[l]:
            _view(h, u, mesh, first, l, 0, len(mesh.coords[l]))[:] = _conserved(*_primitives(case, seed, mesh, l, u.device))
    return h, mesh, first, extra


def _view(h, state, mesh, first, l, at, count):
    """The interiors of ``count`` patches of level l from slot ``at``, in place."""
    nv, m, d = mesh.dim + 2, mesh.n[l] + 2 * NG, mesh.dim
    size = nv * m ** d
    off = h.offset(first[l]) + at * size
    t = state[off:off + count * size].reshape([count, nv] + [m] * d)
    return t[(slice(None), slice(None)) + (slice(NG, -NG),) * d]


def _views(h, state, mesh, first):
    return [_view(h, state, mesh, first, l, 0, len(mesh.coords[l])) for l in range(mesh.nlev) if mesh.coords[l]]


def _net(case, seed):
    """Weights of the predictor (He-normal, small biases) in its flat layout, and
    the normalisation of its inputs."""
    d = case["dim"]
    ci, ch, k = (4, 16, 9) if d == 2 else (5, 8, 27)
    r = np.random.default_rng(3000 + seed)
    w = [r.normal(0, math.sqrt(2 / (ci * k)), ch * ci * k), r.normal(0, 0.05, ch), r.normal(0, math.sqrt(2 / (ch * k)), ch * ch * k),
         r.normal(0, 0.05, ch), r.normal(0, math.sqrt(2 / (ch * k)), ch * k), r.normal(0, 0.05, 1)]
    return np.concatenate(w).astype(np.float32), [1.0] + [0.0] * d + [2.0], [0.3] + [0.2] * d + [4.0]


def _batch(case, seed, device):
    """Normalised fields of a training batch (smooth, with a front) in bfloat16,
    channel-last, and the cells near the front as labels."""
    d, n, t = case["dim"], case["edge"], case["tiles"]
    w, ci = n + 6, (4 if case["dim"] == 2 else 5)
    g = torch.Generator(device=device).manual_seed(4000 + seed)
    axes = [torch.arange(w, device=device, dtype=torch.float32) / w for _ in range(d)]
    ax = torch.meshgrid(*axes, indexing="ij")
    nrm = torch.randn([t, d] + [1] * d, generator=g, device=device)
    s = sum(nrm[:, j] * (ax[j] - 0.5) for j in range(d)) + 0.4 * torch.randn([t] + [1] * d, generator=g, device=device)
    amp = torch.randn([t, ci] + [1] * d, generator=g, device=device)
    slope = torch.randn([t, ci] + [1] * d, generator=g, device=device)
    f = amp * torch.tanh(12.0 * s)[:, None] + slope * s[:, None]
    x = torch.zeros([t] + [w] * d + [4 if d == 2 else 8], device=device)
    x[..., :ci] = f.movedim(1, -1)
    y = (s.abs() < 0.08)[(slice(None),) + (slice(3, -3),) * d]
    return x.to(torch.bfloat16).reshape(t, w ** d, -1), y.to(torch.uint8).reshape(t, n ** d).contiguous()


POS_WEIGHT, RATE = 4.0, 1e-3


def prepare(case, seed):
    kind = case["kind"]
    if kind == "train":
        from paper_2508_05020_amd import amr, workloads

        d = case["dim"]
        cfg = workloads.AMRConfig(name="train", dim=d, base_cells=32, patch_cells=[16], periodic=[True] * d, max_patches=64)
        h = amr.Hierarchy(cfg)
        w, mean, std = _net(case, seed)
        net = amr.Predictor(h, case["edge"], mean, std, pos_weight=POS_WEIGHT, max_batch=case["tiles"])
        net.set_weights(w)
        x, y = _batch(case, seed, h.device)
        return dict(kind=kind, h=h, net=net, x=x.view(torch.int16).contiguous(), y=y, grads=torch.zeros(net.nparams, device=h.device))
    h, mesh, first, extra = _hierarchy(case, seed)
    s = dict(kind=kind, h=h)
    if kind == "step":
        h.set_graph(case["graph"])
        s["dt"] = torch.zeros(1, dtype=F64, device=h.device)
        s["out"] = _views(h, h.state_tensor(0), mesh, first)
    elif kind == "rhs":
        s["rhs"] = h.new_state_like()
        s["out"] = _views(h, s["rhs"], mesh, first)
    elif kind == "tag":
        s["cells"] = case["cells"]   # per-cell tags too, as the predictor's labels need them
    elif kind == "regrid":
        r = np.zeros(h.cfg.max_patches, np.uint8)
        r[[first[l] + mesh.index[l][c] for l, c in extra]] = 1
        s["flags"], s["none"] = r, np.zeros_like(r)
        l, ratio = (extra[0][0], 2 * mesh.n[extra[0][0]] // mesh.n[extra[0][0] + 1]) if extra else (0, 0)
        s["out"] = [_view(h, h.state_tensor(0), mesh, first, l + 1, len(mesh.coords[l + 1]), len(extra) * ratio ** mesh.dim)] if extra else []
    elif kind == "gradient":
        d, nv = mesh.dim, mesh.dim + 2
        g = s["planes"] = torch.zeros(d * d + 1, h.state_doubles // nv, dtype=F64, device=h.device)
        s["out"] = []
        for l in range(mesh.nlev):
            m, count = mesh.n[l] + 2 * NG, len(mesh.coords[l])
            if count:
                off = h.offset(first[l]) // nv
                t = g[:, off:off + count * m ** d].reshape([d * d + 1, count] + [m] * d)
                s["out"].append(t[(slice(None), slice(None)) + (slice(NG, -NG),) * d])
    elif kind == "predict":
        w, mean, std = _net(case, seed)
        count = min(case["tiles"], len(mesh.coords[-1]))
        s["net"] = _predictor(h, mesh.n[-1], mean, std, count)
        s["net"].set_weights(w)
        s["pids"] = [first[-1] + k for k in range(count)]
    return s


def _predictor(h, edge, mean, std, count):
    from paper_2508_05020_amd import amr

    return amr.Predictor(h, edge, mean, std, pos_weight=POS_WEIGHT, max_batch=count)


def run(s):
    kind, h = s["kind"], s["h"]
    if kind == "step":
        h.step(s["dt"])
        return [s["dt"], s["out"]]
    if kind == "rhs":
        h.rhs(0, s["rhs"])
        return s["out"]
    if kind == "tag":
        refine, coarsen, cells = h.tag(0, cell_tags=s["cells"])
        return [refine, coarsen, cells]
    if kind == "regrid":
        made = h.regrid(s["flags"], s["none"])
        gone = h.regrid(s["none"], s["flags"])
        return [made[0], gone[1], s["out"]]
    if kind == "gradient":
        h.velocity_gradient(0, s["planes"])
        return s["out"]
    if kind == "train":
        loss = s["net"].train_step(s["x"], s["y"], RATE, s["grads"])
        return [loss, s["grads"]]
    x = s["net"].gather(0, s["pids"])
    return [x, s["net"].forward(x)]


def work(case):
    """Bytes and operations of one pass: the state read and written once per
    stage, the input tiles and logits once; an edge's interpolation and flux
    once per cell and direction."""
    kind, d = case["kind"], case["dim"]
    nv = d + 2
    if kind == "train":
        n, t = case["edge"], case["tiles"]
        f = t * _net_flops(d, n)
        return dict(bytes=t * ((n + 6) ** d * (8 if d == 2 else 16) + 5 * n ** d), flops=3 * f)
    mesh = Mesh(case)
    cells = mesh.leaf_cells()
    edge = {"weno": nv * 110 + 90, "char": nv * 150 + 200, "central": nv * 5 + 90}[case["scheme"]]
    if kind == "step":
        return dict(bytes=8 * 8 * nv * cells, flops=3 * d * edge * cells)
    if kind == "rhs":
        return dict(bytes=2 * 8 * nv * cells, flops=d * edge * cells)
    if kind == "tag":
        return dict(bytes=8 * nv * cells, flops=(10 + 12 * d) * cells)
    if kind == "regrid":
        new = sum(mesh.n[l] ** d * 2 ** d for l, _ in mesh.extra())
        return dict(bytes=8 * nv * (new + new / 2 ** d), flops=max(1, 100 * new))
    if kind == "gradient":
        return dict(bytes=8 * (d + 1 + d * d + 1) * cells, flops=(4 * d * d + 4 * d) * cells)
    n, t = mesh.n[-1], min(case["tiles"], len(mesh.coords[-1]))
    return dict(bytes=t * (n + 6) ** d * (8 * nv + (8 if d == 2 else 16)) + 4 * t * n ** d, flops=t * _net_flops(d, n))


def _net_flops(d, n):
    ci, ch, k = (4, 16, 9) if d == 2 else (5, 8, 27)
    return 2 * k * (ch * ci * (n + 4) ** d + ch * ch * (n + 2) ** d + ch * n ** d)


# ---------------------------------------------------------------------------
# the same passes from the definitions, in 64 bits on the CPU
# ---------------------------------------------------------------------------
class Flow:
    """State arrays U[l] [P, nv, n, ...] of every level and the operators on them."""

    def __init__(self, case, seed):
        self.case, self.mesh = case, Mesh(case)
        m = self.mesh
        self.d, self.nv, self.scheme = m.dim, m.dim + 2, case["scheme"]
        self.h = [1.0 / c for c in m.cells]
        self.leaf = [m.leaves(l) for l in range(m.nlev)]
        self.map = []
        for l in range(m.nlev):
            a = torch.full([m.np[l]] * self.d, -1, dtype=torch.int64)
            if m.coords[l]:
                c = torch.tensor(m.coords[l]).reshape(-1, self.d)
                a[tuple(c[:, j] for j in reversed(range(self.d)))] = torch.arange(len(c))
            self.map.append(a)
        self.co = [torch.tensor(c, dtype=torch.int64).reshape(-1, self.d) for c in m.coords]
        self.U = [_conserved(*_primitives(case, seed, m, l, "cpu")) for l in range(m.nlev)]

    def wrap(self, l, g):
        N = self.mesh.cells[l]
        return [v % N if self.mesh.periodic else v.clamp(0, N - 1) for v in g]

    def at(self, l, g):
        """Patch (-1 where there is none) and cell within it of in-domain cells g."""
        n = self.mesh.n[l]
        q = [torch.div(v, n, rounding_mode="floor") for v in g]
        k = self.map[l][tuple(reversed(q))]
        loc = 0
        for j in reversed(range(self.d)):
            loc = loc * n + (g[j] - q[j] * n)
        return k, loc

    def pick(self, A, l, g):
        """[nv, K] values of level l at cells g (all present)."""
        k, loc = self.at(l, g)
        assert bool((k >= 0).all())
        return A[l].reshape(A[l].shape[0], A[l].shape[1], -1)[k, :, loc].T

    def prolong(self, A, l, g):
        """MC-limited linear interpolation from the level below; without slopes
        where a child of the coarse cell would have no positive density or pressure."""
        gc = [torch.div(v, 2, rounding_mode="floor") for v in g]
        phi, slopes = self.pick(A, l - 1, gc), []
        for j in range(self.d):
            side = []
            for s in (1, -1):
                q = list(gc)
                q[j] = q[j] + s
                side.append(self.pick(A, l - 1, self.wrap(l - 1, q)))
            a, b = side[0] - phi, phi - side[1]
            mag = torch.minimum(2 * torch.minimum(a.abs(), b.abs()), 0.5 * (a + b).abs())
            slopes.append(torch.where(a * b > 0, torch.sign(a) * mag, torch.zeros_like(a)))
        bad = torch.zeros(phi.shape[1], dtype=torch.bool)
        for sg in itertools.product((-0.25, 0.25), repeat=self.d):
            ch = phi + sum(c * s for c, s in zip(sg, slopes))
            p = self.prims(ch, 0)[-1]
            bad |= ~((ch[0] > 0) & (p > 0))
        val = phi.clone()
        for j in range(self.d):
            val = val + (0.5 * (g[j] % 2).to(F64) - 0.25) * torch.where(bad, torch.zeros_like(phi), slopes[j])
        return val

    def prims(self, U, dim=1):
        """rho, u_j, p along axis ``dim``."""
        u = U.unbind(dim)
        v = [m / u[0] for m in u[1:-1]]
        return [u[0]] + v + [(GAMMA - 1.0) * (u[-1] - 0.5 * sum(m * w for m, w in zip(u[1:-1], v)))]

    def box(self, A, l, sel, ghosts):
        """Patches ``sel`` of level l with ``ghosts[j]`` layers around them in direction j."""
        d, n = self.d, self.mesh.n[l]
        shape = [len(sel)] + [n + 2 * ghosts[j] for j in reversed(range(d))]
        g = []
        for j in range(d):
            v = self.co[l][sel, j:j + 1] * n + torch.arange(-ghosts[j], n + ghosts[j])
            s = [len(sel)] + [1] * d
            s[d - j] = v.shape[1]
            g.append(v.reshape(s).expand(shape).reshape(-1))
        g = self.wrap(l, g)
        k, loc = self.at(l, g)
        flat = A[l].reshape(A[l].shape[0], self.nv, -1)
        out = flat[k.clamp(min=0), :, loc].T.contiguous()
        if bool((miss := k < 0).any()):
            out[:, miss] = self.prolong(A, l, [v[miss] for v in g])
        return out.reshape([self.nv] + shape).transpose(0, 1)

    # -- fluxes ------------------------------------------------------------
    @staticmethod
    def weno(v):
        """Left-biased value from five nodes."""
        a, b, c, d, e = v
        q = ((3 * a - 10 * b + 15 * c) / 8, (-b + 6 * c + 3 * d) / 8, (3 * c + 6 * d - e) / 8)
        s = (13 / 12 * (a - 2 * b + c) ** 2 + 0.25 * (a - 4 * b + 3 * c) ** 2,
             13 / 12 * (b - 2 * c + d) ** 2 + 0.25 * (b - d) ** 2,
             13 / 12 * (c - 2 * d + e) ** 2 + 0.25 * (3 * c - 4 * d + e) ** 2)
        w = [x / (EPS + y) ** 2 for x, y in zip((1 / 16, 10 / 16, 5 / 16), s)]
        return sum(x * y for x, y in zip(w, q)) / sum(w)

    def flux(self, rho, u, p, j):
        E = p / (GAMMA - 1.0) + 0.5 * rho * sum(v * v for v in u)
        U = [rho] + [rho * v for v in u] + [E]
        F = [x * u[j] for x in U]
        F[1 + j] = F[1 + j] + p
        F[-1] = F[-1] + p * u[j]
        return U, F, torch.sqrt(GAMMA * p / rho) + u[j].abs()

    def edges(self, B, j):
        """Rusanov flux at the n + 3 edges of each line along the (last) axis of B [P, nv, ..., n + 8]."""
        n3 = B.shape[-1] - 5
        nodes = lambda x: [x[..., k:k + n3] for k in range(6)]  # noqa: E731
        rho, *u, p = self.prims(B)
        if self.scheme == "char":
            return self.edges_char(B, j, nodes)
        fields = [p, p / rho] + u
        left, right, a, b = [], [], [], []
        for f in fields:
            v = nodes(f)
            a.append(v[2])
            b.append(v[3])
            if self.scheme == "central":
                left.append((9 * (v[2] + v[3]) - v[1] - v[4]) / 16)
                right.append(left[-1])
            else:
                left.append(self.weno(v[:5]))
                right.append(self.weno(v[:0:-1]))
        ok = (left[0] > 0) & (left[1] > 0) & (right[0] > 0) & (right[1] > 0)
        left = [torch.where(ok, x, y) for x, y in zip(left, a)]
        right = [torch.where(ok, x, y) for x, y in zip(right, b)]
        sides = [self.flux(w[0] / w[1], w[2:], w[0], j) for w in (left, right)]
        return self.rusanov(sides)

    @staticmethod
    def rusanov(sides):
        (UL, FL, sl), (UR, FR, sr) = sides
        S = torch.maximum(sl, sr)
        return torch.stack([0.5 * (fl + fr - S * (ur - ul)) for ul, ur, fl, fr in zip(UL, UR, FL, FR)], 1)

    def edges_char(self, B, j, nodes):
        """The same with the eigenvectors of the flux Jacobian at the mean of the two nodes."""
        d, nv = self.d, self.nv
        V = [nodes(x) for x in B.unbind(1)]
        mean = [0.5 * (v[2] + v[3]) for v in V]
        rho, *u, p = self.prims(torch.stack(mean, 1))
        q2 = sum(x * x for x in u)
        c = torch.sqrt(GAMMA * p / rho)
        H = (mean[-1] + p) / rho
        b1 = (GAMMA - 1) / (c * c)
        b2 = 0.5 * b1 * q2
        W = []
        for k in range(6):
            x = [V[v][k] for v in range(nv)]
            s = b1 * (x[-1] - sum(u[i] * x[1 + i] for i in range(d))) + b2 * x[0]
            a = (u[j] * x[0] - x[1 + j]) / c
            W.append([0.5 * (s + a), x[0] - s] + [x[1 + t] - u[t] * x[0] for t in range(d) if t != j] + [0.5 * (s - a)])
        states, ok = [], None
        for side in (0, 1):
            w = []
            for f in range(nv):
                v = [W[k][f] for k in range(6)]
                w.append(self.weno(v[:5] if side == 0 else v[:0:-1]))
            r = w[0] + w[1] + w[-1]
            mom, e, g = [None] * d, H * (w[0] + w[-1]) + u[j] * c * (w[-1] - w[0]) + 0.5 * q2 * w[1], 2
            for t in range(d):
                if t == j:
                    mom[t] = u[j] * r + c * (w[-1] - w[0])
                else:
                    mom[t] = u[t] * r + w[g]
                    e = e + u[t] * w[g]
                    g += 1
            U = [r] + mom + [e]
            pr = self.prims(torch.stack(U, 1))[-1]
            good = (r > 0) & (pr > 0)
            ok = good if ok is None else ok & good
            states.append(U)
        sides = []
        for side in (0, 1):
            U = [torch.where(ok, x, V[v][2 + side]) for v, x in enumerate(states[side])]
            r, *w, pr = self.prims(torch.stack(U, 1))
            sides.append(self.flux(r, w, pr, j))
        return self.rusanov(sides)

    def faces(self, A, l):
        """Face fluxes of every patch of level l: per direction [P, nv, ..., n + 1] with that direction last."""
        out = []
        every = torch.arange(len(self.co[l]))
        for j in range(self.d):
            part = []
            for sel in every.split(max(1, 200_000 // self.mesh.n[l] ** self.d)):
                g = [NG if i == j else 0 for i in range(self.d)]
                F = self.edges(self.box(A, l, sel, g).movedim(1 + self.d - j, -1), j)
                part.append(F[..., 1:-1] - (F[..., :-2] - 2 * F[..., 1:-1] + F[..., 2:]) / 24)
            out.append(torch.cat(part))
        return out

    def rhs(self, A):
        m, d = self.mesh, self.d
        G = [self.faces(A, l) if m.coords[l] else None for l in range(m.nlev)]
        for l in range(m.nlev - 1):
            if not m.coords[l + 1]:
                continue
            n, nf, Nf = m.n[l], m.n[l + 1], m.cells[l + 1]
            for j, side in itertools.product(range(d), (0, 1)):
                off = [0] * d
                off[j] = 2 * side - 1
                ks = [k for k, c in enumerate(m.coords[l]) if c not in m.parents[l] and m.neighbour(l, c, off) in m.parents[l]]
                if not ks:
                    continue
                c = self.co[l][ks]
                F = 2 * (c[:, j] + side) * n
                cj = F % Nf if side else (F - 1) % Nf
                tang = [i for i in reversed(range(d)) if i != j]   # the array order of what is left
                avg = 0
                for o in itertools.product((0, 1), repeat=d - 1):
                    g = [None] * d
                    g[j] = cj.reshape([-1] + [1] * (d - 1))
                    for a, (i, oi) in enumerate(zip(tang, o)):
                        s = [-1] + [1] * (d - 1)
                        s[1 + a] = n
                        g[i] = (2 * (c[:, i:i + 1] * n + torch.arange(n)) + oi).reshape([len(ks)] + s[1:])
                    g = torch.broadcast_tensors(*g)
                    k, _ = self.at(l + 1, list(g))
                    loc = [v % nf for v in g]
                    idx = [loc[i] for i in tang] + [loc[j] + (0 if side else 1)]
                    avg = avg + torch.stack([G[l + 1][j][:, v][(k, *idx)] for v in range(self.nv)], 1)
                G[l][j][ks, ..., n if side else 0] = avg / 2 ** (d - 1)
        out = []
        for l in range(m.nlev):
            r = torch.zeros_like(A[l])
            for j in range(d):
                if G[l] is not None:
                    r -= ((G[l][j][..., 1:] - G[l][j][..., :-1]) / self.h[l]).movedim(-1, 1 + d - j)
            out.append(r)
        return out

    def restrict(self, A):
        m, d = self.mesh, self.d
        for l in range(m.nlev - 1, 0, -1):
            if not m.coords[l]:
                continue
            hn = m.n[l] // 2
            x = A[l]
            for a in range(2, 2 + d):
                x = 0.5 * (x.index_select(a, torch.arange(0, 2 * hn, 2)) + x.index_select(a, torch.arange(1, 2 * hn, 2))) \
                    if x.shape[a] == 2 * hn else x
            shape = [len(self.co[l])] + [hn] * d
            g = []
            for j in range(d):
                s = [len(self.co[l])] + [1] * d
                s[d - j] = hn
                g.append((self.co[l][:, j:j + 1] * hn + torch.arange(hn)).reshape(s).expand(shape).reshape(-1))
            k, loc = self.at(l - 1, g)
            A[l - 1].reshape(A[l - 1].shape[0], self.nv, -1)[k, :, loc] = x.transpose(0, 1).reshape(self.nv, -1).T

    def step(self):
        rate = 0.0
        for l, u in enumerate(self.U):
            if bool(self.leaf[l].any()):
                rho, *v, p = self.prims(u[self.leaf[l]])
                rate = max(rate, float((sum(w.abs() for w in v) + self.d * torch.sqrt(GAMMA * p / rho)).max()) / self.h[l])
        dt, old, cur = CFL / rate, self.U, self.U
        for w in (1.0, 0.25, 2.0 / 3.0):
            R = self.rhs(cur)
            new = [o + w * ((c + dt * r) - o) for o, c, r in zip(old, cur, R)]
            self.restrict(new)
            cur = new
        return dt, cur


def exact(case, seed):
    kind, d = case["kind"], case["dim"]
    torch.set_num_threads(max(1, min(16, torch.get_num_threads())))
    if kind == "tag":
        return None                      # flags only
    if kind == "train":
        return _exact_train(case, seed)
    if kind in ("step", "rhs", "gradient") and Mesh(case).all_cells() * (9 if kind == "step" else 3) > {1: 3e7, 2: 4e7, 3: 1.5e7}[d]:
        return None                      # minutes in plain torch
    f = Flow(case, seed)
    m = f.mesh
    if kind == "step":
        dt, U = f.step()
        return [torch.tensor([dt], dtype=F64), [u for u in U if len(u)]]
    if kind == "rhs":
        R = f.rhs(f.U)
        for l, r in enumerate(R):
            r[~f.leaf[l]] = 0.0
        return [r for r in R if len(r)]
    if kind == "regrid":
        extra = m.extra()
        if not extra:
            return [None, None, []]
        l = extra[0][0]
        n, r = m.n[l + 1], 2 * m.n[l] // m.n[l + 1]
        co = torch.tensor([[a * r + b for a, b in zip(c, reversed(o))] for _, c in extra for o in itertools.product(range(r), repeat=d)])
        shape, g = [len(co)] + [n] * d, []
        for j in range(d):
            s = [len(co)] + [1] * d
            s[d - j] = n
            g.append((co[:, j:j + 1] * n + torch.arange(n)).reshape(s).expand(shape).reshape(-1))
        return [None, None, [f.prolong(f.U, l + 1, g).reshape([f.nv] + shape).transpose(0, 1)]]
    if kind == "gradient":
        out = []
        for l in range(m.nlev):
            if not m.coords[l]:
                continue
            B = f.box(f.U, l, torch.arange(len(f.co[l])), [1] * d)
            rho, *u, _ = f.prims(B)
            diff = lambda x, j: ((x.narrow(d - j, 2, m.n[l]) - x.narrow(d - j, 0, m.n[l])) / (2 * f.h[l]))[  # noqa: E731
                tuple([slice(None)] + [slice(None) if a == d - j else slice(1, -1) for a in range(1, d + 1)])]
            planes = [diff(u[i], j) for i in range(d) for j in range(d)]
            planes.append(torch.sqrt(sum(diff(rho, j) ** 2 for j in range(d))))
            t = torch.stack(planes)
            t[:, ~f.leaf[l]] = 0.0
            out.append(t)
        return out
    w, mean, std = _net(case, seed)
    sel = torch.arange(min(case["tiles"], len(m.coords[-1])))
    x = torch.stack([(v - a) / s for v, a, s in zip(f.prims(f.box(f.U, m.nlev - 1, sel, [3] * d)), mean, std)], 1)
    return [None, _layers(d, x, _weights(d, w)).detach().reshape(len(sel), -1)]


def _weights(d, w):
    ci, ch, k = (4, 16, 9) if d == 2 else (5, 8, 27)
    shapes = [[ch, ci] + [3] * d, [ch], [ch, ch] + [3] * d, [ch], [1, ch] + [3] * d, [1]]
    out, at = [], 0
    for s in shapes:
        size = math.prod(s)
        out.append(torch.from_numpy(w[at:at + size]).to(F64).reshape(s).requires_grad_(True))
        at += size
    return out


def _layers(d, x, w):
    conv = torch.nn.functional.conv2d if d == 2 else torch.nn.functional.conv3d
    a = torch.relu(conv(x, w[0], w[1]))
    a = torch.relu(conv(a, w[2], w[3]))
    return conv(a, w[4], w[5])[:, 0]


def _exact_train(case, seed):
    d, n, t = case["dim"], case["edge"], case["tiles"]
    # the batch itself is made where the timed pass makes it: its random stream is the device's
    x, y = _batch(case, seed, "cuda" if torch.cuda.is_available() else "cpu")
    x = x.cpu().to(F64).reshape([t] + [n + 6] * d + [-1]).movedim(-1, 1)[:, :4 if d == 2 else 5]
    w = _weights(d, _net(case, seed)[0])
    z = _layers(d, x, w).reshape(t, -1)
    y = y.cpu().to(F64)
    sp = torch.nn.functional.softplus
    loss = (POS_WEIGHT * y * sp(-z) + (1 - y) * sp(z)).mean()
    loss.backward()
    return [loss.detach().reshape(1), torch.cat([v.grad.reshape(-1) for v in w])]
