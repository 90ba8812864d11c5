"""The work a user of this framework has it do, as measurable cases over its public entry points.

Three kinds of work: coupled steps of one lattice with a snapshot at the end (``lattice``), batched
parameter sweeps sampled on the device (``sweep``, ``series``), and the surrogate network's forward,
gradient and training calls (``forward``, ``noalloc``, ``gradients``, ``train``).  ``exact`` holds a
plain 64-bit torch version of the same method, written from the method's equations.

All inputs follow from the seed.  Snapshots and series are kept in single precision, as plots and
the network's training take them.
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2209_14889_amd import lb, mlp, surrogate
from paper_2209_14889_amd import workload as wl

NET = list(surrogate.WIDTHS)                    # 5 -> 256 -> 256 -> 256 -> 64
# free-energy coefficients of the closed box and the channel: Table III read in Pa (as paper_case)
FE_PA = dict(alpha=-0.9 / 500.0, beta=1.0 / 500.0, kappa=0.001 / 500.0)


def listed() -> list:
    return [
        # one query of the surrogate: the smallest call there is, all launch latency
        dict(name="forward-1", kind="forward", batch=1, widths="net"),
        # the held-out set of 512 rows in a serving loop that may not allocate
        dict(name="noalloc-512", kind="noalloc", batch=512, widths="net"),
        # screening the parameter space with the trained network
        dict(name="forward-65536", kind="forward", batch=65536, widths="net"),
        # one epoch of the surrogate's training: 14 Adam steps on minibatches of 256 rows
        dict(name="train-256", kind="train", batch=256, steps=14, widths="net"),
        # gradients of a wider network on a ragged batch
        dict(name="gradients-wide-1000", kind="gradients", batch=1000, widths="16,1000,1000,130"),
        # the smallest lattice in use: 64 x 64, random directors, one body
        dict(name="lattice-64", kind="lattice", recipe="c1", nx=64, ny=64, walls=0, fp16=False, bodies=1, steps=500),
        # the paper's own experiment: 250 x 250 closed box, the droplet dragged by the trap
        dict(name="box-250", kind="lattice", recipe="paper", nx=250, ny=250, walls=2, fp16=False, bodies=1, steps=1000),
        # the mid-size single simulation, resident in cache
        dict(name="lattice-512", kind="lattice", recipe="c2", nx=512, ny=512, walls=0, fp16=False, bodies=1, steps=1000),
        # a ragged channel with several bodies, larger than the caches
        dict(name="channel-1400x1001", kind="lattice", recipe="small", nx=1400, ny=1001, walls=1, fp16=False, bodies=3,
             radius=16.0, steps=300),
        # the headline: 2048 x 2048, FP16 storage, eight bodies
        dict(name="lattice-2048-fp16", kind="lattice", recipe="c3", nx=2048, ny=2048, walls=0, fp16=True, bodies=8,
             steps=1000),
        # a parameter sweep: members of uneven sizes in one ensemble, body forces sampled every 64 steps
        dict(name="sweep-64", kind="sweep", members=64, steps=256, every=64),
        # the surrogate's fallback: the full protocol of 32 lattices of 128 x 128, created, run, read
        dict(name="series-32", kind="series", members=32, n=128, steps=4096, every=64),
    ]


def _log_int(rng, lo, hi) -> int:
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng) -> dict:
    kind = rng.choice(["lattice", "lattice", "lattice", "lattice", "sweep", "series", "forward", "noalloc", "train",
                       "gradients"])
    if kind == "lattice":
        nx, ny = _log_int(rng, 24, 1600), _log_int(rng, 24, 1600)
        steps = max(50, min(1000, int(4e8 / (nx * ny))))
        walls = rng.choice([0, 0, 1, 2])
        bodies = rng.choice([0, 1, 1, 2]) if nx >= 48 else rng.choice([0, 1])
        room = min(ny, nx / max(1, bodies)) / 2.0
        return dict(kind=kind, recipe="small", nx=nx, ny=ny, walls=walls, fp16=rng.random() < 0.3, bodies=bodies,
                    radius=round(min(rng.uniform(4.0, 16.0), room - 7.0), 2), steps=steps)
    if kind == "sweep":
        return dict(kind=kind, members=_log_int(rng, 3, 64), steps=rng.choice([128, 192, 256]), every=64)
    if kind == "series":
        return dict(kind=kind, members=_log_int(rng, 2, 48), n=rng.choice([64, 96, 128]), steps=1024, every=64)
    hidden = rng.choice([64, 100, 256, 256, 256, 384])
    widths = ",".join(map(str, [5] + [hidden] * rng.choice([2, 3]) + [rng.choice([16, 64])]))
    if kind == "forward":
        return dict(kind=kind, batch=_log_int(rng, 2, 65536), widths=widths)
    if kind == "noalloc":
        return dict(kind=kind, batch=_log_int(rng, 2, 1365), widths=widths)
    if kind == "train":
        return dict(kind=kind, batch=_log_int(rng, 32, 1024), steps=_log_int(rng, 2, 14), widths=widths)
    return dict(kind=kind, batch=_log_int(rng, 2, 4096), widths=widths)


# -- inputs ---------------------------------------------------------------------------------------

def _lattice(case, seed) -> "wl.Workload":
    rng = np.random.default_rng(seed)
    nx, ny, nb = case["nx"], case["ny"], case["bodies"]
    if case["recipe"] == "c1":
        return wl.c1(seed, nx, ny)
    if case["recipe"] == "c2":
        return wl.c2(seed, nx)
    if case["recipe"] == "c3":
        w = wl.c3(n=nx, n_bodies=nb)                # the workload's own bodies, another director field
        th = math.radians(30.0) + rng.normal(0.0, 0.1, size=(ny, nx))
        w.sims[0].P0 = wl.director_field(th, math.sqrt(0.9))
        return w
    if case["recipe"] == "paper":
        return wl.paper_case(alpha=-float(rng.uniform(0.3, 0.9)), theta0=float(rng.uniform(0.0, math.pi)), n=nx)
    over = FE_PA if case["walls"] else {}
    return wl.small_case(seed, nx, ny, nb, radius=case["radius"], random_dirs=False, D_p=float(rng.uniform(0.001, 0.1)),
                         relax=float(rng.uniform(50.0, 400.0)), pull=5e-5, walls=case["walls"], **over)


def _members(case, seed) -> list:
    return [wl.ensemble_member(i, seed_base=2000 + 1000 * (seed % 100003)) for i in range(case["members"])]


def _series_seeds(case, seed) -> list:
    base = 3000 + 1000 * (seed % 100003)
    return list(range(base, base + case["members"]))


def _widths(case) -> list:
    return NET if case["widths"] == "net" else [int(w) for w in case["widths"].split(",")]


def _net_data(case, seed):
    """Glorot weights with small biases, inputs in [-1, 1], and smooth target series."""
    w, rng = _widths(case), np.random.default_rng(seed)
    p, o = mlp.init_params(w, seed), 0
    for a, b in zip(w[:-1], w[1:]):
        o += a * b
        p[o:o + b] = rng.uniform(-0.1, 0.1, b)
        o += b
    rows = case["batch"] * case.get("steps", 1)
    X = rng.uniform(-1.0, 1.0, (rows, w[0])).astype(np.float32)
    t = np.linspace(0.0, 1.0, w[-1])
    Y = np.sin(np.outer(1.0 + X[:, 0], 3.0 * t) + X[:, 1:2]) * (1.5 + X[:, 2:3]) + 0.3 * X[:, 3:4] * X[:, 4:5]
    return w, p, X, Y.astype(np.float32)


def prepare(case, seed):
    kind = case["kind"]
    if kind == "lattice":
        w = _lattice(case, seed)
        return dict(case=case, sim=lb.Sim(w, lb.make_options(precision=int(case["fp16"]), graph_chunk=100)))
    if kind == "sweep":
        return dict(case=case, sim=lb.Sim(_members(case, seed), lb.make_options(graph_chunk=case["every"])))
    if kind == "series":
        return dict(case=case, seeds=_series_seeds(case, seed))
    w, p, X, Y = _net_data(case, seed)
    s = dict(case=case, widths=w, X=torch.from_numpy(X).cuda(), Y=torch.from_numpy(Y).cuda())
    if kind == "noalloc":
        s["params"] = torch.from_numpy(p).cuda()
        s["out"] = torch.empty((case["batch"], w[-1]), dtype=torch.float32, device="cuda")
    else:
        s["net"] = mlp.MLP(w, case["batch"])
        s["net"].set_params(p)
        s["loss"] = torch.zeros(1, dtype=torch.float32, device="cuda")
    torch.cuda.synchronize()
    return s


# -- one pass -------------------------------------------------------------------------------------

def run(state):
    case = state["case"]
    kind = case["kind"]
    if kind == "lattice":
        sim = state["sim"]
        sim.step(case["steps"])
        out = {k: torch.from_numpy(v).to(torch.float32) for k, v in sim.fields().items()}
        if case["bodies"]:
            out["nodes"] = [torch.from_numpy(r).to(torch.float32) for r in sim.nodes()]
        return out
    if kind == "sweep":
        sim = state["sim"]
        samples = torch.empty((case["steps"] // case["every"], case["members"], 8), dtype=torch.float64, device="cuda")
        for row in samples:
            sim.step(case["every"])
            sim.body_forces_device(row)
        sim.sync()
        return samples.to(torch.float32)
    if kind == "series":
        _, y = surrogate.simulate(state["seeds"], n=case["n"], steps=case["steps"], every=case["every"])
        return torch.from_numpy(y).to(torch.float32)
    if kind == "noalloc":
        mlp.forward_noalloc(state["widths"], state["params"], state["X"], state["out"])
        return state["out"]
    net = state["net"]
    if kind == "forward":
        return net.forward(state["X"])
    if kind == "gradients":
        loss, g = net.gradients(state["X"], state["Y"])
        return {"loss": np.float32(loss), "gradients": g}
    b = case["batch"]
    for k in range(case["steps"]):
        net.train_step(state["X"][k * b:(k + 1) * b], state["Y"][k * b:(k + 1) * b], 2e-4, state["loss"])
    return {"params": net.get_params(), "loss": state["loss"]}


def work(case) -> dict:
    kind = case["kind"]
    if kind in ("lattice", "sweep", "series"):
        # a site update reads and writes 9 populations, 3 stresses and 2 polarizations once, and takes
        # about 570 operations
        per = 76 if case.get("fp16") else 112
        if kind == "lattice":
            sites, out = case["nx"] * case["ny"], 10 * 4 * case["nx"] * case["ny"]
        elif kind == "sweep":
            sites, out = sum(s.nx * s.ny for s in _members(case, 0)), 0
        else:
            sites, out = case["members"] * case["n"] ** 2, 0
        return {"bytes": per * sites * case["steps"] + out, "flops": 570 * sites * case["steps"]}
    w = _widths(case)
    n = sum(a * b + b for a, b in zip(w[:-1], w[1:]))
    rows = case["batch"] * case.get("steps", 1)
    io, products = 4 * rows * (w[0] + w[-1]), 2 * rows * sum(a * b for a, b in zip(w[:-1], w[1:]))
    if kind in ("forward", "noalloc"):
        return {"bytes": 4 * n + io, "flops": products}
    back = 3 * products - 2 * rows * w[0] * w[1]      # the first layer's inputs take no gradient
    if kind == "gradients":
        return {"bytes": 8 * n + io, "flops": back}
    return {"bytes": 24 * n * case["steps"] + io, "flops": back}


# -- the same in 64 bits --------------------------------------------------------------------------

CX = (0, 1, 0, -1, 0, 1, -1, -1, 1)
CY = (0, 0, 1, 0, -1, 1, 1, -1, -1)
WQ = (4 / 9,) + (1 / 9,) * 4 + (1 / 36,) * 4
OPP = (0, 3, 4, 1, 2, 7, 8, 5, 6)


def _closure(p_clamp: float, dev, n: int = 4096):
    """a2 / s and a4 / s^2 of the von Mises closure at s = i p_clamp^2 / n, with a_m = I_m(k) / I_0(k)
    and I_1(k) / I_0(k) = sqrt(s)."""
    s = torch.arange(1, n + 3, dtype=torch.float64, device=dev) * (p_clamp ** 2 / n)
    p = s.sqrt()
    lo, hi = torch.zeros_like(p), torch.full_like(p, 1e4)
    for _ in range(80):
        k = 0.5 * (lo + hi)
        less = torch.special.i1e(k) < p * torch.special.i0e(k)
        lo, hi = torch.where(less, k, lo), torch.where(less, hi, k)
    th = torch.arange(2048, dtype=torch.float64, device=dev) * (2.0 * math.pi / 2048)
    w = torch.exp(k[:, None] * (torch.cos(th) - 1.0))
    z = w.sum(1)
    a2 = (w * torch.cos(2.0 * th)).sum(1) / z / s
    a4 = (w * torch.cos(4.0 * th)).sum(1) / z / (s * s)
    first = lambda v: torch.tensor([v], dtype=torch.float64, device=dev)  # noqa: E731
    return torch.cat([first(0.5), a2]), torch.cat([first(1.0 / 24.0), a4]), n / p_clamp ** 2


class _Lattices:
    """Independent lattices, their sites in one flat array, stepped in 64 bits."""

    def __init__(self, sims, dev="cuda"):
        self.dev, self.sims = dev, sims
        one = len(sims) == 1
        f64 = dict(dtype=torch.float64, device=dev)
        sizes = [s.nx * s.ny for s in sims]
        off = np.concatenate([[0], np.cumsum(sizes)])
        self.n = int(off[-1])

        def site(get):   # a coefficient per site (a plain number for a single lattice)
            v = [float(get(s.params)) for s in sims]
            return v[0] if one else torch.repeat_interleave(torch.tensor(v, **f64), torch.tensor(sizes, device=dev))

        self.omega = site(lambda q: 1.0 / q["tau"])
        self.inv_eta, self.D = site(lambda q: 1.0 / q["eta_p"]), site(lambda q: q["D_p"])
        self.xi, self.kappa, self.Gamma = site(lambda q: q["xi"]), site(lambda q: q["kappa"]), site(lambda q: q["Gamma"])
        self.alpha, self.beta = site(lambda q: q["alpha"]), site(lambda q: q["beta"])
        self.eon = site(lambda q: float(q.get("ericksen", 1)))
        K = [site(lambda q, i=i: q["Kx"][i]) for i in range(4)]
        self.KA, self.KB = K[0] - 2 * K[1] - 4 * K[3] + K[2], K[0] - K[2]
        self.iso = ((3 * K[0] + 2 * K[1] + 4 * K[3] + 3 * K[2]) / 8, (K[0] + 6 * K[1] - 4 * K[3] + K[2]) / 8,
                    (K[0] - 2 * K[1] + 4 * K[3] + K[2]) / 4)
        self.clamp = float(sims[0].params["P_clamp"])
        self.A2, self.A4, self.per_s = _closure(self.clamp, dev)
        nbr, sgn, pull = [], [], [[] for _ in range(9)]
        for s, o in zip(sims, off[:-1]):
            walls = int(s.params.get("walls", 0))
            y, x = torch.meshgrid(torch.arange(s.ny, device=dev), torch.arange(s.nx, device=dev), indexing="ij")
            here = (int(o) + y * s.nx + x).reshape(-1)

            def at(dx, dy):
                X, Y = x + dx, y + dy
                out = torch.zeros_like(X, dtype=torch.bool)
                if walls:
                    out = out | (Y < 0) | (Y >= s.ny)
                if walls == 2:
                    out = out | (X < 0) | (X >= s.nx)
                return (int(o) + (Y % s.ny) * s.nx + X % s.nx).reshape(-1), out.reshape(-1)

            row, sg = [], []
            for dx, dy in ((1, 0), (-1, 0), (0, 1), (0, -1)):
                i, out = at(dx, dy)
                row.append(torch.where(out, here, i))              # mirror ghost
                sg.append(torch.where(out, -1.0, 1.0).to(torch.float64))   # no-slip: negated ghost
            nbr.append(torch.stack(row))
            sgn.append(torch.stack(sg))
            for m in range(9):
                i, out = at(-CX[m], -CY[m])
                pull[m].append(torch.where(out, OPP[m] * self.n + here, m * self.n + i))
        self.nbr = torch.cat(nbr, 1)
        sg = torch.cat(sgn, 1)
        self.sgn = None if bool((sg == 1.0).all()) else sg
        self.pull = torch.cat([torch.cat(q) for q in pull])
        plane = lambda a, c: torch.from_numpy(np.asarray(a, np.float64).reshape(c, -1))  # noqa: E731
        self.P = torch.cat([plane(s.P0, 2) for s in sims], 1).to(dev)
        self.sig = torch.zeros((3, self.n), **f64)
        self.h = torch.tensor(WQ, **f64)[:, None].repeat(1, self.n)
        self.t = 0
        self._bodies(off, f64)

    def _bodies(self, off, f64):
        bs = [(b, s, int(o)) for s, o in zip(self.sims, off[:-1]) for b in s.bodies]
        self.bodies, self.nb = bs, len(bs)
        if not bs:
            return
        cnt = [b.R.shape[0] for b, _, _ in bs]
        st = np.concatenate([[0], np.cumsum(cnt)])
        self.start = st
        t = lambda v: torch.tensor(np.asarray(v, np.float64), **f64)  # noqa: E731
        i = lambda v: torch.tensor(np.asarray(v, np.int64), device=self.dev)  # noqa: E731
        self.R = t(np.concatenate([b.R for b, _, _ in bs]))
        loc = [np.arange(c) for c in cnt]
        self.nxt = i(np.concatenate([o + (a + 1) % c for o, a, c in zip(st, loc, cnt)]))
        self.prv = i(np.concatenate([o + (a - 1) % c for o, a, c in zip(st, loc, cnt)]))
        self.own = i(np.repeat(np.arange(self.nb), cnt))
        self.cnt = t(cnt)
        self.ks, self.eps = t([b.k_spring for b, _, _ in bs])[self.own], t([b.eps_angle for b, _, _ in bs])[self.own]
        self.leq = t([b.l_eq for b, _, _ in bs])[self.own]
        self.force = t([b.pull for b, _, _ in bs])
        self.bnx, self.bny = i([s.nx for _, s, _ in bs])[self.own], i([s.ny for _, s, _ in bs])[self.own]
        self.boff = i([o for _, _, o in bs])[self.own]

    # fields ------------------------------------------------------------------------------------
    def _n4(self, f):
        return f[..., self.nbr[0]], f[..., self.nbr[1]], f[..., self.nbr[2]], f[..., self.nbr[3]]

    def _div(self, a):   # divergence of a stress given as (xx, xy, yx, yy) planes
        return (0.5 * (a[0][self.nbr[0]] - a[0][self.nbr[1]]) + 0.5 * (a[1][self.nbr[2]] - a[1][self.nbr[3]]),
                0.5 * (a[2][self.nbr[0]] - a[2][self.nbr[1]]) + 0.5 * (a[3][self.nbr[2]] - a[3][self.nbr[3]]))

    def _mol(self, P, n4):   # molecular field
        a = self.alpha + self.beta * (P[0] * P[0] + P[1] * P[1])
        return a * P - self.kappa * (n4[0] + n4[1] + n4[2] + n4[3] - 4.0 * P)

    def _force(self):
        s = self.sig
        Fx, Fy = self._div((s[0], s[2], s[2], s[1]))
        self.fp = (Fx.clone(), Fy.clone())
        n4 = self._n4(self.P)
        P, H = self.P, self._mol(self.P, n4)
        dx, dy = 0.5 * (n4[0] - n4[1]), 0.5 * (n4[2] - n4[3])
        anti = -0.5 * (P[0] * H[1] - H[0] * P[1])
        sym = 0.5 * self.xi * (P[0] * H[1] + H[0] * P[1])
        g = self.kappa * (dx * dy).sum(0)
        E = (self.xi * P[0] * H[0] - self.kappa * (dx * dx).sum(0), anti + sym - g, sym - anti - g,
             self.xi * P[1] * H[1] - self.kappa * (dy * dy).sum(0))
        ex, ey = self._div(E)
        Fx, Fy = Fx + self.eon * ex, Fy + self.eon * ey
        if self.nb:
            self.fn = self._node_forces()
            idx, w = self._kernel(self.R)
            Fx.index_add_(0, idx.reshape(-1), (self.fn[:, 0:1] * w).reshape(-1))
            Fy.index_add_(0, idx.reshape(-1), (self.fn[:, 1:2] * w).reshape(-1))
        return Fx, Fy

    def _moments(self, Fx, Fy):
        h = self.h
        rho = h.sum(0)
        jx = h[1] - h[3] + h[5] - h[6] - h[7] + h[8]
        jy = h[2] - h[4] + h[5] + h[6] - h[7] - h[8]
        return rho, (jx + 0.5 * Fx) / rho, (jy + 0.5 * Fy) / rho

    def _stiff(self):
        """The anisotropic stiffness as a function applying it to plain components (xx, yy, xy)."""
        P, smax = self.P, self.clamp ** 2
        s = P[0] * P[0] + P[1] * P[1]
        u = torch.clamp(s, max=smax) * self.per_s
        j = torch.clamp(u.to(torch.int64), 1, self.A2.numel() - 3)
        t = u - j
        c = (-t * (t - 1) * (t - 2) / 6, (t + 1) * (t - 1) * (t - 2) / 2, -(t + 1) * t * (t - 2) / 2,
             (t + 1) * t * (t - 1) / 6)
        A2 = sum(c[m] * self.A2[j + (m - 1)] for m in range(4))
        A4 = sum(c[m] * self.A4[j + (m - 1)] for m in range(4))
        r = torch.where(s > smax, smax / torch.clamp(s, min=1e-300), torch.ones_like(s))
        d, e = P[0] * P[0] - P[1] * P[1], 2.0 * P[0] * P[1]
        X1, Y1 = A4 * r * r * (d * d - e * e) * self.KA, A4 * r * r * 2.0 * d * e * self.KA
        X2, Y2 = A2 * r * d * self.KB, A2 * r * e * self.KB
        C11, C12, C33 = self.iso[0] + X1 / 8 + X2 / 2, self.iso[1] - X1 / 8, self.iso[2] - X1 / 4
        C22, C13, C23 = C11 - X2, (Y1 + 2.0 * Y2) / 4, (2.0 * Y2 - Y1) / 4
        return lambda a, b, c_: (C11 * a + C12 * b + C13 * c_, C12 * a + C22 * b + C23 * c_,
                                 0.5 * (C13 * a + C23 * b) + C33 * c_)

    def step(self):
        Fx, Fy = self._force()
        rho, ux, uy = self._moments(Fx, Fy)
        uu, uF, guo = ux * ux + uy * uy, ux * Fx + uy * Fy, 1.0 - 0.5 * self.omega
        post = torch.empty_like(self.h)
        for m in range(9):
            cu, cF = CX[m] * ux + CY[m] * uy, CX[m] * Fx + CY[m] * Fy
            eq = WQ[m] * rho * (1.0 + 3.0 * cu + 4.5 * cu * cu - 1.5 * uu)
            post[m] = self.h[m] - self.omega * (self.h[m] - eq) + guo * WQ[m] * (3.0 * (cF - uF) + 9.0 * cu * cF)
        self.h = post.reshape(-1)[self.pull].reshape(9, -1)
        del post
        v = torch.stack([ux, uy])
        e, w, n, s = self._n4(v)
        if self.sgn is not None:
            e, w, n, s = e * self.sgn[0], w * self.sgn[1], n * self.sgn[2], s * self.sgn[3]
        gx, gy = 0.5 * (e - w), 0.5 * (n - s)          # d_x v, d_y v
        psi = (gx[0], gy[1], 0.5 * (gx[1] + gy[0]))
        om = 0.5 * (gx[1] - gy[0])
        C = self._stiff()

        def rhs_sigma(X):
            n4 = self._n4(X)
            c = C(*(psi[q] - self.inv_eta * X[q] for q in range(3)))
            turn = (2.0 * om * X[2], -2.0 * om * X[2], om * (X[1] - X[0]))
            adv = ux * 0.5 * (n4[0] - n4[1]) + uy * 0.5 * (n4[2] - n4[3])
            return torch.stack(c) - torch.stack(turn) - adv + self.D * (n4[0] + n4[1] + n4[2] + n4[3] - 4.0 * X)

        def rhs_P(Y):
            n4 = self._n4(Y)
            adv = ux * 0.5 * (n4[0] - n4[1]) + uy * 0.5 * (n4[2] - n4[3])
            turn = torch.stack([om * Y[1], -om * Y[0]])
            flow = torch.stack([psi[0] * Y[0] + psi[2] * Y[1], psi[2] * Y[0] + psi[1] * Y[1]])
            return self.xi * flow - adv - turn - self.Gamma * self._mol(Y, n4)

        r = rhs_sigma(self.sig)
        self.sig = self.sig + 0.5 * (r + rhs_sigma(self.sig + r))
        r = rhs_P(self.P)
        self.P = self.P + 0.5 * (r + rhs_P(self.P + r))
        if self.nb:
            k1 = self._interp(self.R, ux, uy)
            self.R = self.R + 0.5 * (k1 + self._interp(self.R + k1, ux, uy))
        self.t += 1

    def fields(self) -> dict:
        Fx, Fy = self._force()
        rho, ux, uy = self._moments(Fx, Fy)
        s = self.sims[0]
        planes = (rho, ux, uy, *self.sig, *self.P, *self.fp)
        return {k: p.reshape(s.ny, s.nx) for k, p in zip(lb.FIELDS, planes)}

    # bodies ------------------------------------------------------------------------------------
    def _kernel(self, R):
        """Site indices (nodes, 16) and cosine-kernel weights of every node's 4 x 4 footprint."""
        i0 = torch.floor(R).to(torch.int64) - 1
        k = torch.arange(4, device=self.dev)
        xs, ys = i0[:, 0:1] + k, i0[:, 1:2] + k
        wx = 0.25 * (1.0 + torch.cos(0.5 * math.pi * (R[:, 0:1] - xs)))
        wy = 0.25 * (1.0 + torch.cos(0.5 * math.pi * (R[:, 1:2] - ys)))
        ys = ys % self.bny[:, None] * self.bnx[:, None] + self.boff[:, None]
        return ((ys[:, :, None] + (xs % self.bnx[:, None])[:, None, :]).reshape(-1, 16),
                (wy[:, :, None] * wx[:, None, :]).reshape(-1, 16))

    def _interp(self, R, ux, uy):
        idx, w = self._kernel(R)
        return torch.stack([(ux[idx] * w).sum(1), (uy[idx] * w).sum(1)], 1)

    def _com(self):
        c = torch.zeros((self.nb, 2), dtype=torch.float64, device=self.dev).index_add_(0, self.own, self.R)
        return c / self.cnt[:, None]

    def _node_forces(self):
        R = self.R
        e2, e1 = R[self.nxt] - R, R[self.prv] - R
        l2, l1 = e2.norm(dim=1, keepdim=True), e1.norm(dim=1, keepdim=True)
        k, leq = self.ks[:, None], self.leq[:, None]
        f = k * (l2 - leq) / l2 * e2 + k * (l1 - leq) / l1 * e1
        cg = (e1 * e2).sum(1, keepdim=True) / (l1 * l2)
        d1 = self.eps[:, None] * (e2 / (l1 * l2) - cg * e1 / (l1 * l1))
        d2 = self.eps[:, None] * (e1 / (l1 * l2) - cg * e2 / (l2 * l2))
        f = f + d1 + d2 - d1[self.nxt] - d2[self.prv]
        sig = lambda z: 0.5 * (1.0 + math.tanh(0.5 * z))  # noqa: E731
        soft = lambda z: max(z, 0.0) + math.log1p(math.exp(-abs(z)))  # noqa: E731
        share = torch.zeros((self.nb, 2), dtype=torch.float64)
        com = None
        for q, (b, _, _) in enumerate(self.bodies):
            on = sig((self.t - b.t_on) / b.width) - sig((self.t - b.t_off) / b.width) if b.width > 0 else 1.0
            share[q, 0], share[q, 1] = on * b.pull[0], on * b.pull[1]
            if b.trap:
                tr = b.trap
                com = self._com().cpu() if com is None else com
                u1, u2 = (self.t - tr["t1"]) / tr["w"], (self.t - tr["t2"]) / tr["w"]
                T = tr["t2"] - tr["t1"]
                along = tr["w"] / T * (soft(u1) - soft(u2)) if T > 0 else 0.0
                kt = tr["k"] * (sig(u1) - sig(u2))
                share[q, 0] += kt * (tr["x0"] + tr["dx"] * along - com[q, 0])
                share[q, 1] += kt * (tr["y0"] + tr["dy"] * along - com[q, 1])
        return f + (share.to(self.dev) / self.cnt[:, None])[self.own]

    def observables(self):
        """Per body: site-sum restoring force, centre of mass, total node force, area-weighted force."""
        s = self.sig
        fx, fy = self._div((s[0], s[2], s[2], s[1]))
        com, fn = self._com(), self._node_forces()
        tot = torch.zeros((self.nb, 2), dtype=torch.float64, device=self.dev).index_add_(0, self.own, fn)
        out = torch.empty((self.nb, 8), dtype=torch.float64, device=self.dev)
        out[:, 2:4], out[:, 4:6] = com, tot
        box = torch.stack([torch.stack([self.R[a:b].amin(0), self.R[a:b].amax(0)])
                           for a, b in zip(self.start[:-1], self.start[1:])]).cpu().numpy()
        for q, (_, spec, o) in enumerate(self.bodies):
            R = self.R[self.start[q]:self.start[q + 1]]
            (x0, y0), (x1, y1) = np.floor(box[q, 0]) - 1, np.ceil(box[q, 1]) + 1
            X = torch.arange(x0, x1 + 1, dtype=torch.float64, device=self.dev)
            Y = torch.arange(y0, y1 + 1, dtype=torch.float64, device=self.dev)
            site = o + (Y.long() % spec.ny)[:, None] * spec.nx + (X.long() % spec.nx)[None, :]
            A, B = R.roll(1, 0), R
            ya, yb = A[:, 1], B[:, 1]
            # inside by the even-odd rule
            cross = (ya > Y[:, None]) != (yb > Y[:, None])
            xc = (B[:, 0] - A[:, 0]) * (Y[:, None] - ya) / torch.where(yb == ya, torch.ones_like(ya), yb - ya) + A[:, 0]
            inside = ((cross[:, None, :] & (X[None, :, None] < xc[:, None, :])).sum(2) % 2).double()
            # area of every cell inside, by Green's theorem: sum over edges of (clamp(x) - x_left) dy
            lo = torch.maximum(torch.minimum(ya, yb), Y[:, None] - 0.5)
            hi = torch.minimum(torch.maximum(ya, yb), Y[:, None] + 0.5)
            dy = torch.clamp(hi - lo, min=0.0) * torch.sign(yb - ya)
            slope = (B[:, 0] - A[:, 0]) / torch.where(yb == ya, torch.ones_like(ya), yb - ya)
            xl, xh = A[:, 0] + slope * (lo - ya), A[:, 0] + slope * (hi - ya)
            L = X[None, :, None] - 0.5
            xl, xh = (xl[:, None, :] - L), (xh[:, None, :] - L)
            G = lambda z: 0.5 * torch.clamp(z, 0.0, 1.0) ** 2 + torch.clamp(z - 1.0, min=0.0)  # noqa: E731
            near = (xh - xl).abs() < 1e-6
            mean = torch.where(near, torch.clamp(0.5 * (xl + xh), 0.0, 1.0),
                               (G(xh) - G(xl)) / torch.where(near, torch.ones_like(xl), xh - xl))
            area = (mean * dy[:, None, :]).sum(2)
            area = area * torch.sign(area.sum())
            out[q, 0], out[q, 1] = (inside * fx[site]).sum(), (inside * fy[site]).sum()
            out[q, 6], out[q, 7] = (area * fx[site]).sum(), (area * fy[site]).sum()
        return out


def _exact_net(case, seed):
    w, p, X, Y = _net_data(case, seed)
    X, Y = torch.from_numpy(X).cuda().double(), torch.from_numpy(Y).cuda().double()
    p = torch.from_numpy(p).cuda().double()

    def forward(p, x):
        o = 0
        for q, (a, b) in enumerate(zip(w[:-1], w[1:])):
            x = x @ p[o:o + a * b].view(b, a).T + p[o + a * b:o + a * b + b]
            o += a * b + b
            x = torch.tanh(x) if q < len(w) - 2 else x
        return x

    def loss_grad(p, x, y):
        p = p.detach().requires_grad_(True)
        loss = (((forward(p, x) - y) ** 2).sum(1) / (y ** 2).sum(1)).mean()
        return float(loss.detach()), torch.autograd.grad(loss, p)[0]

    if case["kind"] in ("forward", "noalloc"):
        return forward(p, X)
    if case["kind"] == "gradients":
        loss, g = loss_grad(p, X, Y)
        return {"loss": np.float64(loss), "gradients": g}
    m, v, b, loss = torch.zeros_like(p), torch.zeros_like(p), case["batch"], 0.0
    for k in range(case["steps"]):
        loss, g = loss_grad(p, X[k * b:(k + 1) * b], Y[k * b:(k + 1) * b])
        m, v = 0.9 * m + 0.1 * g, 0.999 * v + 0.001 * g * g
        p = p - 2e-4 * (m / (1 - 0.9 ** (k + 1))) / ((v / (1 - 0.999 ** (k + 1))).sqrt() + 1e-8)
    return {"params": p, "loss": torch.tensor([loss], dtype=torch.float64)}


def exact(case, seed):
    kind = case["kind"]
    if kind == "lattice":
        r = _Lattices(_lattice(case, seed).sims)
        for _ in range(case["steps"]):
            r.step()
        out = r.fields()
        if case["bodies"]:
            out["nodes"] = [r.R[a:b] for a, b in zip(r.start[:-1], r.start[1:])]
        return out
    if kind in ("sweep", "series"):
        sims = _members(case, seed) if kind == "sweep" else [wl.surrogate_member(s, case["n"])
                                                             for s in _series_seeds(case, seed)]
        r, rows = _Lattices(sims), []
        for _ in range(case["steps"] // case["every"]):
            for _ in range(case["every"]):
                r.step()
            rows.append(r.observables())
        return torch.stack(rows) if kind == "sweep" else torch.stack([q[:, 6] for q in rows], 1)
    return _exact_net(case, seed)
