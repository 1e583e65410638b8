"""The work that a user of this framework has it do, as cases to time.

Every case goes through the public entry points (`Simulation`, `Batch`, `Mlp`)
as the programs of this repository do: a chunk of time steps followed by what
such a program reads between chunks, a chunk of the drag-data ensemble with its
training rows, inference and training steps of the drag closure.  Sizes and
physical parameters are those of `inputs.workload`, `validation.py`,
`ensemble.py` and `closure_pipeline.py`, or scaled from them.

`listed` gives the named cases, `draw` further ones of the same ranges,
`prepare` what a program holds before the call, `run` one pass, `work` the
bytes and operations of a pass, and `exact` the same outputs in binary64 from
plain torch.
"""
import functools
import math

import numpy as np
import torch

from paper_1011_2613_amd import binding, ensemble, inputs

BYTES = {"fp64": 8, "fp32s": 4, "fp16s": 2}
# lattice rows per tile that the ensemble's autotuner keeps, as a program reads
# them from its JSON cache
TILE_ROWS = {32: 16, 48: 4, 64: 1, 96: 1}
# a tolerance that no box meets: every box advances through the whole chunk
NEVER = 1e-300


def _suspension(name, base, shape, radius, count, storage, steps, read, **over):
    """A suspension case from the parameters of the named workload `base`."""
    w = inputs.workload(base)
    case = {"kind": "suspension", "dim": w.dim, "nx": shape[0], "ny": shape[1],
            "nz": shape[2] if w.dim == 3 else 1, "wall": w.wall_y, "tau": w.tau, "radius": radius,
            "count": count, "rho_ratio": w.rho_ratio, "samples": w.samples, "kn": w.kn,
            "restitution": w.restitution, "v0": w.v0, "force_x": w.fluid_force[0],
            "force_y": w.fluid_force[1], "accel_y": w.particle_accel[1], "fixed": False,
            "storage": storage, "lists": 0, "steps": steps, "read": read}
    case.update(over)
    if name:
        case["name"] = name
    return case


def _sphere(name, d, steps):
    """One fixed sphere of diameter d in a periodic cube of edge 2.5 d, driven
    to Re_p 0.2 (the resolution study of validation.py)."""
    edge, tau = int(round(2.5 * d)), 1.0
    nu = (tau - 0.5) / 3.0
    c = math.pi * d ** 3 / 6.0 / edge ** 3
    K = 1.0 / (1.0 - 1.7601 * c ** (1.0 / 3.0) + c - 1.5593 * c * c)
    g = 3.0 * math.pi * nu * d * (0.2 * nu / d) * K / edge ** 3
    return _suspension(name, "C3", (edge, edge, edge), d / 2.0, 1, "fp64", steps, "forces", wall=False,
                       tau=tau, rho_ratio=1.0, kn=0.0, v0=0.0, force_x=g, force_y=0.0, accel_y=0.0,
                       fixed=True)


def listed():
    c2, c3 = inputs.workload("C2"), inputs.workload("C3")
    return [
        # a program that looks at its particles after every step: 16 discs, one step
        _suspension("coupled_2d", "C1", (256, 256), 6.0, 16, "fp64", 1, "particles", v0=5.0e-3),
        # the same small suspension left to run: a chunk of steps between two records
        _suspension("run_2d", "C1", (256, 256), 6.0, 16, "fp64", 100, "stats", v0=5.0e-3),
        # the resolution study at d/l = 32: one large fixed sphere, a chunk between two drag checks
        _sphere("sphere_cube", 32, 50),
        # an odd-sized dense channel with the paper's neighbour lists, binary32 storage
        _suspension("ragged_3d", "C3", (101, 163, 77), 5.3, 310, "fp32s", 50, "stats", lists=100),
        # the 2D suspension of the benchmark, 8192 x 2048 with 21 361 discs
        _suspension("suspension_2d", "C2", c2.shape, c2.radius, c2.count, "fp64", 50, "stats"),
        # the 3D suspension of the benchmark, 192 x 756 x 192 with 8 317 spheres
        _suspension("suspension_3d", "C3", c3.shape, c3.radius, c3.count, "fp64", 50, "stats"),
        # the same with half-precision storage
        _suspension("suspension_3d_fp16", "C3", c3.shape, c3.radius, c3.count, "fp16s", 50, "stats"),
        # an eighth of the paper's fully periodic 3D domain, binary32 storage (the largest)
        _suspension("paper_3d_fp32", "P3", (512, 252, 512), 5.0, 16128, "fp32s", 20, "stats"),
        # a chunk of a 64-box drag-data ensemble and its training rows
        {"name": "ensemble", "kind": "ensemble", "boxes": 64, "steps": 100},
        # the closure on a million particles, and on the spheres of one suspension
        {"name": "closure_rows", "kind": "infer", "rows": 1 << 20},
        {"name": "closure_spheres", "kind": "infer", "rows": c3.count},
        # one optimiser step of the closure's training
        {"name": "closure_training", "kind": "train", "rows": 4096},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(("2d", "2d", "3d", "3d", "3d", "sphere", "ensemble", "infer", "train"))
    if kind == "sphere":
        return _sphere(None, rng.randint(6, 32), rng.randint(10, 50))
    if kind == "ensemble":
        return {"kind": "ensemble", "boxes": _log(rng, 4, 64), "steps": 2 * rng.randint(10, 50)}
    if kind == "infer":
        return {"kind": "infer", "rows": _log(rng, 1, 1 << 20)}
    if kind == "train":
        return {"kind": "train", "rows": _log(rng, 32, 4096)}
    if kind == "2d":
        base, shape = rng.choice(("C1", "C2")), (_log(rng, 64, 8192), _log(rng, 64, 2048))
    else:
        base, shape = "C3", (_log(rng, 32, 256), _log(rng, 32, 512), _log(rng, 32, 192))
    dim = len(shape)
    radius = rng.uniform(3.0, 7.0)
    phi = rng.uniform(0.03, 0.15)
    count = max(1, min(20000, inputs.solid_fraction_count(dim, shape, radius, phi)))
    rho = inputs.workload(base).rho_ratio
    # the stiffness of a ten-step contact, as in the named workloads
    m = rho * (math.pi * radius ** 2 if dim == 2 else 4.0 / 3.0 * math.pi * radius ** 3)
    kn = (math.pi ** 2 + math.log(0.9) ** 2) * 0.5 * m / 100.0
    nodes = shape[0] * shape[1] * (shape[2] if dim == 3 else 1)
    steps = max(1, min(100, 2 * 10 ** 8 // nodes, rng.randint(1, 100)))
    return _suspension(None, base, shape, radius, count, rng.choice(("fp64", "fp32s", "fp16s")), steps,
                       rng.choice(("stats", "forces", "particles")), wall=rng.random() < 0.5, kn=kn,
                       v0=5.0e-3, lists=rng.choice((0, 0, 100)))


def _workload(case, seed):
    shape = (case["nx"], case["ny"], case["nz"])[: case["dim"]]
    return inputs.Workload("case", case["dim"], shape, case["tau"], case["wall"], case["radius"],
                           case["count"], case["rho_ratio"], case["samples"], case["kn"],
                           case["restitution"], case["steps"], seed=seed + 11, v0=case["v0"],
                           fluid_force=(case["force_x"], case["force_y"], 0.0),
                           particle_accel=(0.0, case["accel_y"], 0.0), fixed=case["fixed"])


@functools.lru_cache(maxsize=8)
def _sampled(count):
    return ensemble.sample_boxes(count, 4)


def _boxes(case, seed):
    """The ensemble's boxes: edges, sphere counts and forcing of one drawing,
    every box's spheres shifted by a seeded vector (a periodic box, so other
    places between the nodes) and its forcing scaled by a seeded factor."""
    rng = np.random.default_rng(seed)
    out = []
    for b in _sampled(case["boxes"]):
        shift, scale = rng.uniform(0.0, b["edge"], 3), rng.uniform(0.8, 1.2)
        pos = np.mod(b["pos"] + shift, b["edge"])
        pos[pos >= b["edge"]] = 0.0
        out.append(dict(b, pos=pos, fluid_force=tuple(scale * a for a in b["fluid_force"]),
                        init_velocity=tuple(scale * a for a in b["init_velocity"])))
    return out


def _closure_data(case, seed):
    """Parameters, normaliser, raw inputs and targets of the closure."""
    rng = np.random.default_rng(seed)
    params = inputs.mlp_initial_params(seed + 3)
    for _, b in params:
        b[:] = 0.05 * rng.standard_normal(b.shape)
    mu = rng.uniform(-1.0, 1.0, 40).astype(np.float32)
    sd = rng.uniform(0.3, 2.0, 40).astype(np.float32)
    n = case["rows"]
    z = rng.standard_normal((n, 40), dtype=np.float32)
    if case["kind"] == "infer":
        return params, (mu, sd, mu - 3.0 * sd, mu + 3.0 * sd), mu + sd * z, None
    return params, None, z, (np.sin(z[:, 0]) + 0.3 * z[:, 1] * z[:, 2]).astype(np.float32)


def prepare(case, seed):
    if case["kind"] == "suspension":
        w = _workload(case, seed)
        sim = binding.simulation_for(w, storage=case["storage"], with_particles=False)
        if case["lists"]:
            sim.set_neighbour_list(case["lists"])
        sim.set_particles(*w.particles())
        return case, sim
    if case["kind"] == "ensemble":
        batch = binding.Batch(_boxes(case, seed), samples=4)
        for edge in sorted(set(batch.edges)):
            batch.set_tile_rows(edge, TILE_ROWS[edge])
        return case, batch
    params, norm, X, y = _closure_data(case, seed)
    mlp = binding.Mlp(max_batch=4096 if case["kind"] == "train" else 64)
    mlp.set_params(binding.mlp_pack(params))
    if norm is not None:
        mlp.set_normaliser(*norm)
    X = torch.as_tensor(X, device="cuda:0")
    return case, mlp, X, None if y is None else torch.as_tensor(y, device="cuda:0")


STATS = ("mass", "fluid_velocity", "particle_velocity", "mean_drag")


def run(state):
    case, obj = state[:2]
    if case["kind"] == "suspension":
        obj.step(case["steps"])
        # what is read between two chunks: a record of the suspension's time
        # series, the drag or the drag and the particles; and the flow field
        if case["read"] == "stats":
            st = obj.stats()
            return [st[k] for k in STATS], obj.particles(), obj.macro_device()
        return obj.forces(), obj.particles() if case["read"] == "particles" else (), obj.macro_device()
    if case["kind"] == "ensemble":
        obj.run_steady(case["steps"], NEVER, case["steps"])
        return obj.get_drag(), obj.mean_velocity()
    if case["kind"] == "infer":
        return obj.infer(state[2])
    loss = obj.train_step(state[2], state[3], 1e-3)
    return loss, obj.get_params()


def work(case):
    if case["kind"] == "suspension":
        nodes = case["nx"] * case["ny"] * case["nz"]
        Q = 9 if case["dim"] == 2 else 19
        # every step reads and writes the populations; the field reads them
        # once more and is written; about 12 operations per population
        # (moments, equilibrium, relaxation, force)
        moved = 2 * Q * BYTES[case["storage"]] * nodes * case["steps"]
        moved += nodes * (Q * BYTES[case["storage"]] + 8 * (1 + case["dim"]))
        return {"bytes": moved, "flops": 12.0 * Q * nodes * case["steps"]}
    if case["kind"] == "ensemble":
        nodes = sum(b["edge"] ** 3 for b in _sampled(case["boxes"]))
        return {"bytes": 2 * 19 * 4 * nodes * case["steps"], "flops": 12.0 * 19 * nodes * case["steps"]}
    n, par = case["rows"], binding.MLP_NPARAMS
    if case["kind"] == "infer":
        return {"bytes": n * (160 + 4 + 1) + 4 * par, "flops": 2.0 * n * par}
    # forward, input and weight gradients; parameters and both moments updated
    return {"bytes": n * (160 + 4) + 7 * 4 * par, "flops": 6.0 * n * par}


# ------------------------------------------------------- plain binary64 reference
def _device():
    return "cuda:0" if torch.cuda.is_available() else "cpu"


class _Reference:
    """The method (LBGK, immersed moving boundary, soft-sphere contacts) in
    binary64 on whole arrays, from rest or a uniform velocity."""

    def __init__(self, dim, shape, tau, wall, force, accel, samples, kn, restitution, parts, u0=(0.0, 0.0, 0.0)):
        self.dev = _device()
        self.dim, self.tau, self.wall, self.S, self.kn = dim, tau, wall, samples, kn
        self.n = list(shape) + [1] * (3 - dim)
        self.N = int(np.prod(self.n))
        rng3 = [-1, 0, 1]
        self.c = [(x, y, z) for x in rng3 for y in rng3 for z in (rng3 if dim == 3 else [0])
                  if abs(x) + abs(y) + abs(z) <= 2]
        wt = ({0: 4 / 9, 1: 1 / 9, 2: 1 / 36} if dim == 2 else {0: 1 / 3, 1: 1 / 18, 2: 1 / 36})
        self.w = [wt[abs(x) + abs(y) + abs(z)] for x, y, z in self.c]
        self.opp = [self.c.index((-x, -y, -z)) for x, y, z in self.c]
        self.force, self.accel = force, accel
        le = math.log(restitution)
        self.ce = -2.0 * le / math.sqrt(math.pi ** 2 + le ** 2)
        t = lambda a: torch.as_tensor(np.array(a, dtype=np.float64), device=self.dev)  # noqa: E731
        self.x, self.v, self.om, self.R, rho, fixed = (t(a) for a in parts)
        if dim == 2:
            self.m = rho * math.pi * self.R ** 2
            self.I = 0.5 * self.m * self.R ** 2
        else:
            self.m = rho * (4.0 / 3.0) * math.pi * self.R ** 3
            self.I = 0.4 * self.m * self.R ** 2
        self.free = (fixed == 0).double()[:, None]
        one = torch.ones(self.N, dtype=torch.float64, device=self.dev)
        u = [one * a for a in u0]
        self.f = torch.stack([self._eq(i, one, u) for i in range(len(self.c))])
        self.F = torch.zeros_like(self.x)
        self.T = torch.zeros_like(self.x)
        self.eps = torch.zeros(self.N, dtype=torch.float64, device=self.dev)
        self.near = None

    def _dot(self, i, u):
        s = 0.0
        for a in range(3):
            if self.c[i][a]:
                s = s + self.c[i][a] * u[a]
        return s

    def _eq(self, i, rho, u):
        cu = self._dot(i, u)
        uu = u[0] * u[0] + u[1] * u[1] + u[2] * u[2]
        return self.w[i] * rho * (1.0 + 3.0 * cu + 4.5 * cu * cu - 1.5 * uu)

    def _moments(self, f):
        rho = f.sum(0)
        j = [sum(self.c[i][a] * f[i] for i in range(len(self.c)) if self.c[i][a]) for a in range(self.dim)]
        return rho, [a / rho for a in j] + [torch.zeros_like(rho)] * (3 - self.dim)

    def _cover(self):
        """Covered (particle, node) pairs: particle, node, samples inside, offset."""
        P = len(self.R)
        ext = int(math.floor(2.0 * float(self.R.max()) + 1.0)) + 1
        out = []
        step = max(1, 4_000_000 // ext ** self.dim)
        ar = torch.arange(ext, device=self.dev)
        for p0 in range(0, P, step):
            p = torch.arange(p0, min(P, p0 + step), device=self.dev)
            lo = torch.ceil(self.x[p] - self.R[p, None] - 0.5).long()
            d, node = [], []
            for a in range(3):
                k = lo[:, a, None] + ar[None] if a < self.dim else torch.zeros_like(lo[:, :1])
                node.append(k)
                d.append(k.double() - (self.x[p, a, None] if a < self.dim else 0.0))
            shape = (len(p), node[0].shape[1], node[1].shape[1], node[2].shape[1])
            full = lambda a, v: v.reshape(len(p), *[-1 if b == a else 1 for b in range(3)]).expand(shape)  # noqa: E731
            cnt = torch.zeros(shape, dtype=torch.int32, device=self.dev)
            off = [(k + 0.5) / self.S - 0.5 for k in range(self.S)]
            R2 = (self.R[p] ** 2).reshape(-1, 1, 1, 1)
            for ox in off:
                for oy in off:
                    s = full(0, (d[0] + ox) ** 2) + full(1, (d[1] + oy) ** 2)
                    for oz in (off if self.dim == 3 else (None,)):
                        cnt += (s if oz is None else s + full(2, (d[2] + oz) ** 2)) <= R2
            if self.wall:
                cnt *= ((full(1, node[1]) >= 0) & (full(1, node[1]) < self.n[1])).int()
            idx = torch.nonzero(cnt.reshape(-1)).reshape(-1)
            at = [full(a, node[a]).reshape(-1)[idx] % self.n[a] for a in range(3)]
            out.append((p[:, None, None, None].expand(shape).reshape(-1)[idx],
                        at[0] + self.n[0] * (at[1] + self.n[1] * at[2]), cnt.reshape(-1)[idx].double(),
                        torch.stack([full(a, d[a]).reshape(-1)[idx] for a in range(3)], 1)))
        return [torch.cat([o[k] for o in out]) for k in range(4)]

    def _pair(self, d):
        for a in range(self.dim):
            if not (a == 1 and self.wall):
                L = float(self.n[a])
                d[..., a] -= L * torch.round(d[..., a] / L)
        return d

    def _contacts(self):
        P, Fc = len(self.R), torch.zeros_like(self.x)
        if self.near is None:
            # pairs that could touch while no particle moves a lattice unit
            got = []
            for p0 in range(0, P, 1024):
                d = self._pair(self.x[p0:p0 + 1024, None] - self.x[None])
                reach = self.R[p0:p0 + 1024, None] + self.R[None] + 2.0
                i, j = torch.nonzero((d * d).sum(-1) < reach * reach, as_tuple=True)
                got.append(torch.stack([i + p0, j], 1)[i + p0 != j])
            self.near = torch.cat(got)
        i, j = self.near[:, 0], self.near[:, 1]
        d = self._pair(self.x[i] - self.x[j])
        dist = torch.sqrt((d * d).sum(-1))
        k = torch.nonzero(self.R[i] + self.R[j] - dist > 0).reshape(-1)
        i, j, d, dist = i[k], j[k], d[k], dist[k]
        nrm = d / dist[:, None]
        me = self.m[i] * self.m[j] / (self.m[i] + self.m[j])
        vn = ((self.v[i] - self.v[j]) * nrm).sum(-1)
        mag = self.kn * (self.R[i] + self.R[j] - dist) - self.ce * torch.sqrt(me * self.kn) * vn
        Fc.index_add_(0, i, mag[:, None] * nrm)
        if self.wall:
            eta = self.ce * torch.sqrt(self.m * self.kn)
            for side, gap in ((1.0, self.x[:, 1] + 0.5), (-1.0, self.n[1] - 0.5 - self.x[:, 1])):
                over = self.R - gap
                mag = self.kn * over - eta * side * self.v[:, 1]
                Fc[:, 1] += torch.where(over > 0, side * mag, torch.zeros_like(mag))
        return Fc

    def step(self):
        Q, N, dim = len(self.c), self.N, self.dim
        cg = [sum(c[a] * self.force[a] for a in range(3)) for c in self.c]
        p, node, cnt, off = self._cover() if len(self.R) else (None,) * 4
        rho, u = self._moments(self.f)
        covered = None
        if p is not None:
            tot = torch.zeros(N, dtype=torch.float64, device=self.dev).index_add_(0, node, cnt)
            covered = torch.nonzero(tot).reshape(-1)
            slot = torch.empty(N, dtype=torch.long, device=self.dev)
            slot[covered] = torch.arange(len(covered), device=self.dev)
            vel = self.v[p] + torch.linalg.cross(self.om[p], off)
            V = torch.zeros(len(covered), 3, dtype=torch.float64, device=self.dev)
            V.index_add_(0, slot[node], cnt[:, None] * vel)
            tc = tot[covered]
            V = [V[:, a] / tc if a < dim else torch.zeros_like(tc) for a in range(3)]
            eps = torch.clamp(tc / self.S ** dim, max=1.0)
            beta = eps * (self.tau - 0.5) / ((1.0 - eps) + (self.tau - 0.5))
            fc, rc, uc = self.f[:, covered], rho[covered], [a[covered] for a in u]
            q = torch.zeros(len(covered), 3, dtype=torch.float64, device=self.dev)
            new = torch.empty_like(fc)
            for i in range(Q):
                o = self.opp[i]
                Om = fc[o] - fc[i] + self._eq(i, rc, V) - self._eq(o, rc, uc)
                new[i] = (fc[i] - (1.0 - beta) / self.tau * (fc[i] - self._eq(i, rc, uc)) + beta * Om
                          + 3.0 * self.w[i] * rc * cg[i])
                for a in range(dim):
                    q[:, a] += self.c[i][a] * beta * Om
            self.eps = torch.zeros_like(rho)
            self.eps[covered] = eps
        post = torch.empty_like(self.f)
        for i in range(Q):
            post[i] = self.f[i] - (self.f[i] - self._eq(i, rho, u)) / self.tau + 3.0 * self.w[i] * rho * cg[i]
        if covered is not None:
            post[:, covered] = new
            t = (cnt / tot[node])[:, None] * q[slot[node]]
            self.F = torch.zeros_like(self.x).index_add_(0, p, -t)
            self.T = torch.zeros_like(self.x).index_add_(0, p, -torch.linalg.cross(off, t))
            total = self.F + self._contacts() + self.m[:, None] * torch.as_tensor(self.accel, device=self.dev,
                                                                                  dtype=torch.float64)
            self.v = self.v + self.free * total / self.m[:, None]
            self.om = self.om + self.free * self.T / self.I[:, None]
            x = self.x + self.free * self.v
            for a in range(dim):
                if not (a == 1 and self.wall):
                    x[:, a] = torch.where(x[:, a] < 0, x[:, a] + self.n[a], x[:, a])
                    x[:, a] = torch.where(x[:, a] >= self.n[a], x[:, a] - self.n[a], x[:, a])
            self.x = x
        grid = (self.n[2], self.n[1], self.n[0])
        for i, (cx, cy, cz) in enumerate(self.c):
            moved = torch.roll(post[i].reshape(grid), (cz, cy, cx), (0, 1, 2))
            if self.wall and cy:
                row = 0 if cy > 0 else self.n[1] - 1
                moved[:, row] = post[self.opp[i]].reshape(grid)[:, row]
            self.f[i] = moved.reshape(-1)

    def fields(self):
        shape = (self.n[2], self.n[1], self.n[0])[3 - self.dim:]
        rho, u = self._moments(self.f)
        return rho.reshape(shape), torch.stack(u[: self.dim]).reshape((self.dim,) + shape)

    def stats(self):
        rho, u = self._moments(self.f)
        fluid = (1.0 - self.eps) * rho
        vf = torch.stack([(fluid * a).sum() for a in u]) / fluid.sum()
        vp = (self.m[:, None] * self.v).sum(0) / self.m.sum()
        return [float(rho.sum()), vf, vp, self.F.mean(0)]


def _exact_closure(case, seed):
    params, norm, X, y = _closure_data(case, seed)
    t = lambda a: torch.as_tensor(np.array(a), device=_device()).double()  # noqa: E731
    layers = [[t(a.astype(np.float32)).requires_grad_(y is not None) for a in pair] for pair in params]
    h = t(X)
    if norm is not None:
        mu, sd, lo, hi = norm
        h = (h - t(mu)) / t(sd)
    for k, (W, b) in enumerate(layers):
        h = h @ W.T + b
        if k < 3:
            h = h * torch.sigmoid(h)
    if y is None:
        return h[:, 0], ((X < lo) | (X > hi)).any(1).astype(np.uint8)
    loss = ((h[:, 0] - t(y)) ** 2).mean()
    flat = [a for pair in layers for a in pair]
    grads = torch.autograd.grad(loss, flat)
    # the first Adam step: both moments start at zero
    new = [p.detach() - 1e-3 * g / (g.abs() + 1e-8) for p, g in zip(flat, grads)]
    return float(loss), torch.cat([a.reshape(-1) for a in new]).cpu().numpy()


def exact(case, seed):
    if case["kind"] in ("infer", "train"):
        return _exact_closure(case, seed)
    if case["kind"] == "ensemble":
        forces, means = [], []
        for b in _boxes(case, seed):
            n = len(b["pos"])
            parts = (b["pos"], np.zeros((n, 3)), np.zeros((n, 3)), np.full(n, b["radius"]), np.ones(n), np.ones(n))
            ref = _Reference(3, (b["edge"],) * 3, b["tau"], False, b["fluid_force"], (0.0,) * 3, 4, 0.0, 0.9,
                             parts, u0=b["init_velocity"])
            for _ in range(case["steps"]):
                ref.step()
            rho, u = ref.fields()
            forces.append(ref.F.cpu().numpy())
            means.append((rho * u).reshape(3, -1).mean(1).cpu().numpy())
        return (np.concatenate(forces), None), np.array(means)
    w = _workload(case, seed)
    ref = _Reference(w.dim, w.shape, w.tau, w.wall_y, w.fluid_force, w.particle_accel, w.samples, w.kn,
                     w.restitution, w.particles())
    for _ in range(case["steps"]):
        ref.step()
    arrays = [a.cpu().numpy() for a in (ref.x, ref.v, ref.om)]
    if case["read"] == "stats":
        return ref.stats(), arrays, ref.fields()
    return (ref.F.cpu().numpy(), ref.T.cpu().numpy()), arrays if case["read"] == "particles" else (), ref.fields()
