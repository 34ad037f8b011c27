"""The work that a user of this library has it do, as cases of one pass each.

Every case is a dict of plain values.  `listed()` names the standing ones,
`draw(rng)` gives another of the same ranges, `prepare(case, seed)` makes
what a program holds before the call (inputs from the seed, the context with
its fibers, the network), `run(state)` makes one pass through the public
entry points, `work(case)` counts the bytes and operations a pass cannot do
without, and `exact(case, seed)` gives the outputs of the first pass in 64
bits from plain torch, without this library.

Kinds of case:
  shear     a shear cell with free fibers, advanced and read back (the flow
            fields on the device, the fibers' record of the pass)
  coarse    the same with under-resolved fibers and the trained closure
  sediment  one spherocylinder falling in a box closed by free-slip walls
  tumble    two forced spherocylinders in a periodic box with momentum
            stabilization
  batch     independent one-fiber cells in one launch, their features sampled
            every few steps and their records read at the end: how training
            data for the closure are made
  sbf       the slender-body model: time steps of M fibers
  fit       the closure network: gradient over the data, one epoch, prediction
"""
import math
import os

import numpy as np
import torch

from paper_1503_06869_amd import closure, lbm, sbf, scenarios, validation

NET = os.path.join(os.path.dirname(os.path.abspath(closure.__file__)), "closure_net.npz")
ESZ = {"f32": 4, "f16": 2, "bf16": 2, "f64": 8}


def listed():
    return [
        # a program that looks at the fiber after every step: launch latency
        dict(name="cell_32_each_step", kind="shear", n=32, nz=32, fibers=1, lmin=12.0, lmax=20.0, storage="f32",
             wall_u=0.005, steps=1),
        # the single-fiber cell of the tumbling-period runs, sampled every 200 steps
        dict(name="cell_32", kind="shear", n=32, nz=32, fibers=1, lmin=12.0, lmax=20.0, storage="f32", wall_u=0.005,
             steps=200),
        # a ragged mid-size cell in BF16 storage (odd edges, few fibers)
        dict(name="cell_odd_bf16", kind="shear", n=93, nz=121, fibers=10, lmin=16.0, lmax=32.0, storage="bf16",
             wall_u=0.01, steps=50),
        # the main workload of bench.py, FP32 and FP16 storage
        dict(name="shear_256_f32", kind="shear", n=256, nz=256, fibers=64, lmin=24.0, lmax=40.0, storage="f32",
             wall_u=0.01, steps=20),
        dict(name="shear_256_f16", kind="shear", n=256, nz=256, fibers=64, lmin=24.0, lmax=40.0, storage="f16",
             wall_u=0.01, steps=20),
        # many under-resolved fibers with the trained closure (bench.py's learned-coarse form)
        dict(name="coarse_128_closure", kind="coarse", n=128, fibers=200, closure=True, steps=40),
        # the wall-effect box of the sedimentation validation
        dict(name="sediment_160", kind="sediment", nxy=160, nz=1200, aspect=8, orientation="sidewise", storage="f32",
             steps=20),
        # the tumbling validation at its full size: the largest lattice
        dict(name="tumble_576", kind="tumble", n=576, aspect=12, storage="f32", steps=6),
        # 512 uneven cells in one launch (bench.py's batched form) with feature sampling
        dict(name="batch_512", kind="batch", cases=512, lo=24, hi=64, storage="f32", steps=40, sample=10),
        # the slender-body tumbling pair: small solves, latency
        dict(name="sbf_pair", kind="sbf", m=2, modes=5, nq=16, tol=1e-12, dt=10.0, steps=20),
        # the sedimenting cloud of bench.py, fibers apart (a shorter time step
        # keeps them so over a long run)
        dict(name="sbf_cloud_1024", kind="sbf", m=1024, modes=5, nq=16, tol=1e-10, dt=1.0, steps=2),
        # training of the closure network
        dict(name="fit_8192", kind="fit", samples=8192, batch=256),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["shear", "shear", "shear", "coarse", "sediment", "tumble", "batch", "sbf", "sbf", "fit"])
    if kind == "shear":
        n, nz = _log(rng, 26, 288), _log(rng, 26, 288)
        lmax = min(40.0, 0.55 * min(n, nz))
        most = max(1, min(64, int(n * n * nz / 60000.0)))
        return dict(kind="shear", n=n, nz=nz, fibers=_log(rng, 1, most), lmin=round(0.6 * lmax, 2), lmax=round(lmax, 2),
                    storage=rng.choice(["f32", "f32", "f16", "bf16", "f64"]), wall_u=rng.choice([0.005, 0.01]),
                    steps=rng.choice([1, 7, 20, 50]))
    if kind == "coarse":
        n = _log(rng, 48, 144)
        return dict(kind="coarse", n=n, fibers=_log(rng, 4, max(5, min(200, int(n ** 3 / 10000.0)))),
                    closure=rng.random() < 0.7, steps=rng.choice([5, 20, 41]))
    if kind == "sediment":
        return dict(kind="sediment", nxy=_log(rng, 64, 224), nz=_log(rng, 128, 1200), aspect=rng.choice([4, 6, 8, 10, 12]),
                    orientation=rng.choice(["lengthwise", "sidewise"]), storage=rng.choice(["f32", "f32", "f16"]),
                    steps=rng.choice([5, 13, 20]))
    if kind == "tumble":
        return dict(kind="tumble", n=_log(rng, 128, 480), aspect=rng.choice([10, 12, 14]),
                    storage=rng.choice(["f32", "f32", "f16", "bf16"]), steps=rng.choice([3, 6, 11]))
    if kind == "batch":
        lo = rng.randint(24, 32)
        return dict(kind="batch", cases=_log(rng, 6, 448), lo=lo, hi=rng.randint(lo, 64),
                    storage=rng.choice(["f32", "f32", "f16"]), steps=rng.choice([10, 20, 33]), sample=rng.choice([5, 10]))
    if kind == "sbf":
        m = _log(rng, 2, 900)
        return dict(kind="sbf", m=m, modes=rng.choice([3, 5, 5, 7]), nq=rng.choice([9, 16, 16]), tol=1e-10,
                    dt=10.0 if m == 2 else 1.0, steps=20 if m < 8 else 2)
    n = _log(rng, 500, 8000)
    return dict(kind="fit", samples=n, batch=rng.choice([64, 100, 256, 512]))


# ------------------------------------------------------------------ inputs
def _scene(case, seed):
    """The lattice, physics and fibers of a single-lattice case."""
    k = case["kind"]
    if k == "shear":
        sc = scenarios.many_fibers(seed=seed, n=case["n"], nz=case["nz"], n_fibers=case["fibers"],
                                   wall_u=case["wall_u"], length=(case["lmin"], case["lmax"]))
        args = dict(tau=sc.tau, wall_u=sc.wall_u, init_couette=True, storage=case["storage"])
    elif k == "coarse":
        sc = scenarios.learned_coarse(seed=seed, n=case["n"], n_fibers=case["fibers"])
        args = dict(tau=sc.tau, wall_u=sc.wall_u, init_couette=True)
    if k in ("shear", "coarse"):
        fibers = [dict(X=f.X, q=f.q, length=f.length, radius=f.radius, density_ratio=f.density_ratio, V=f.V, W=f.W)
                  for f in sc.fibers]
        return (sc.nx, sc.ny, sc.nz), args, fibers
    g = np.random.default_rng(seed)
    r, L = validation.R_CELLS, case["aspect"] * validation.R_CELLS
    tilt = lambda t: (lambda v: v / np.linalg.norm(v))(np.asarray(t) + 0.05 * g.standard_normal(3))  # noqa: E731
    body = dict(length=L, radius=r, shape="spherocylinder")
    if k == "sediment":
        nxy, nz = case["nxy"], case["nz"]
        F = validation.lattice_force(validation.SED_FORCE, validation.DX, validation.dt())
        X = [0.5 * (nxy - 1) + g.uniform(-2, 2), 0.5 * (nxy - 1) + g.uniform(-2, 2), min(100 * r - 0.5, nz / 3.0)]
        q = scenarios.quat_from_axis(tilt((0, 0, 1) if case["orientation"] == "lengthwise" else (1, 0, 0)))
        args = dict(tau=validation.TAU, storage=case["storage"], x_walls="free-slip", y_walls="free-slip",
                    z_free_slip=True)
        return (nxy, nxy, nz), args, [dict(body, X=np.array(X), q=q, force=(0.0, 0.0, F),
                                           density_ratio=validation.RHO_P / validation.RHO_F)]
    n, c = case["n"], 0.5 * (case["n"] - 1)
    F = validation.lattice_force(validation.TUMBLE_FORCE[case["aspect"]])
    dist = g.uniform(14.8, 16.0)
    args = dict(tau=validation.TAU, storage=case["storage"], z_periodic=True, stabilize=True, contact_k=10.0 * F,
                contact_range=2.0)
    fibers = [dict(body, X=np.array([c + 0.5 * s * dist, c, c]) + g.uniform(-0.5, 0.5, 3),
                   q=scenarios.quat_from_axis(tilt((0, 0, 1))), force=(0.0, 0.0, F),
                   density_ratio=validation.TUMBLE_RHO_P / validation.RHO_F) for s in (-1.0, 1.0)]
    return (n, n, n), args, fibers


def _batch_cases(case, seed):
    return scenarios.batched_cases(seed=seed, n_cases=case["cases"], edge=(case["lo"], case["hi"]))


def _sbf_scene(case, seed):
    if case["m"] == 2:      # the tumbling pair, tilted a little
        g = np.random.default_rng(seed)
        return scenarios.sbf_pair(dist=g.uniform(14.0, 18.0), tilt=g.uniform(0.0, 0.2))
    # a cloud whose fibers do not touch (the model holds from about a radius
    # apart): those closer than 2.5 radii to an earlier one are left out
    m = case["m"]
    sc = scenarios.sbf_cloud(seed=seed, m=m + m // 8 + 4)
    half, keep = 0.5 * sc.length * sc.p, []
    for i in range(len(sc.X)):
        d2 = np.sum((sc.X[keep] - sc.X[i]) ** 2, axis=1) if keep else np.zeros(0)
        near = [keep[j] for j in np.flatnonzero(d2 < (1.25 * sc.length) ** 2)]
        if all(scenarios.segment_distance(sc.X[i] - half[i], 2 * half[i], sc.X[j] - half[j], 2 * half[j])
               >= 2.5 * sc.eps * sc.length for j in near):
            keep.append(i)
    keep = keep[:m]
    sc.X, sc.p, sc.F, sc.M = sc.X[keep], sc.p[keep], sc.F[keep], sc.M[keep]
    return sc


def _fit_data(case, seed):
    """Features and targets with the ranges of the sampled flow: O(0.1 .. 1)
    relative velocities with unequal spreads, smooth targets with noise."""
    g = np.random.default_rng(seed)
    n = case["samples"]
    spread = 0.05 + np.abs(g.standard_normal(lbm.MLP_IN)) * 0.3
    z = g.standard_normal((n, 12))
    X = (z @ g.standard_normal((12, lbm.MLP_IN)) / 3.0 + 0.2 * g.standard_normal((n, lbm.MLP_IN))) * spread
    Y = 0.1 * np.tanh(z @ g.standard_normal((12, lbm.MLP_OUT)) / 3.0) + 0.01 * g.standard_normal((n, lbm.MLP_OUT))
    X = X.astype(np.float32)
    norm = closure.make_norm(X, Y)
    T = (Y / norm.out_scale).astype(np.float32)
    fan = math.sqrt(6.0 / lbm.MLP_IN)
    w = np.concatenate([g.uniform(-fan, fan, 64 * 247), np.zeros(64), g.uniform(-0.3, 0.3, 64 * 64), np.zeros(64),
                        g.uniform(-0.03, 0.03, 6 * 64), np.zeros(6)]).astype(np.float32)
    return X, T, norm, w


def prepare(case, seed):
    k = case["kind"]
    if k in ("shear", "coarse", "sediment", "tumble"):
        (nx, ny, nz), args, fibers = _scene(case, seed)
        s = dict(case=case, done=0)
        s["ctx"] = g = lbm.Context(nx, ny, nz, **args)
        for f in fibers:
            g.add_fiber(**f)
        if case.get("closure"):
            s["net"], _ = closure.load(NET)
            g.set_closure(s["net"])
        dt = torch.float64 if case.get("storage") == "f64" else torch.float32
        s["rho"] = torch.empty((nz, ny, nx), dtype=dt, device="cuda")
        s["u"] = torch.empty((3, nz, ny, nx), dtype=dt, device="cuda")
        return s
    if k == "batch":
        b = lbm.Batch(_batch_cases(case, seed), storage=case["storage"])
        b.autotune(trial_steps=4)
        return dict(case=case, done=0, batch=b)
    if k == "sbf":
        sc = _sbf_scene(case, seed)
        g = sbf.SBF(case["m"], sc.length, sc.eps, nmodes=case["modes"], nq=case["nq"], gmres_tol=case["tol"])
        g.set_fibers(sc.X, sc.p, sc.F, sc.M)
        return dict(case=case, sbf=g)
    X, T, norm, w = _fit_data(case, seed)
    m = lbm.Mlp(seed=0)
    m.set_params(w)
    m.set_norm(norm.in_mean, norm.in_inv_std, norm.out_scale, norm.env_min, norm.env_max)
    x, t = torch.tensor(X, device="cuda"), torch.tensor(T, device="cuda")
    return dict(case=case, net=m, x=x, t=t, y=torch.empty_like(t), epoch=0)


def run(state):
    case = state["case"]
    k, n = case["kind"], case.get("steps")
    if k == "batch":
        b, feats, left = state["batch"], [], n
        while left > 0:
            feats.append(b.features())
            b.step(min(case["sample"], left))
            left -= case["sample"]
        hist = np.stack([b.history(c, state["done"], n) for c in range(b.ncases)])
        state["done"] += n
        return {"features": np.stack(feats), "history": hist}
    if k == "sbf":
        g = state["sbf"]
        g.step(n, case["dt"])
        X, p = g.state()
        V, W = g.velocities()
        return {"X": X, "p": p, "V": V, "W": W}
    if k == "fit":
        m, x, t, y = state["net"], state["x"], state["t"], state["y"]
        ns = x.shape[0]
        loss, grad = m.loss_grad(x.data_ptr(), t.data_ptr(), ns)
        state["epoch"] += 1
        losses = m.train(x.data_ptr(), t.data_ptr(), ns, 1, case["batch"], 1e-3, shuffle_seed=state["epoch"])
        m.forward(x.data_ptr(), ns, y.data_ptr())
        return {"loss": loss, "grad": grad, "losses": losses, "weights": m.params()[0], "y": y}
    g = state["ctx"]
    g.step(n)
    hist = g.history(state["done"], n)
    state["done"] += n
    g.fields_to_device(state["rho"].data_ptr(), state["u"].data_ptr())
    return {"history": hist, "rho": state["rho"], "u": state["u"]}


# ------------------------------------------------------------------ what a pass cannot do without
def work(case):
    k = case["kind"]
    if k == "sbf":
        # per step: the moments, and 8 products with the distinct entries of
        # the symmetric matrix (the iterations of a solve that starts from
        # the extrapolated solution)
        m, P1, Q = case["m"], case["modes"] + 1, 3 * case["nq"]
        D = 3 * m * P1
        pairs = m * (m - 1) / 2
        prods = 8
        return dict(bytes=case["steps"] * prods * D * (D + 1) / 2 * 8.0,
                    flops=case["steps"] * (pairs * (Q * Q * (33 + 15 * P1) + 21.0 * Q * P1 * P1) + prods * 2.0 * D * D))
    if k == "fit":
        par, ns = 20422, case["samples"]
        batches = -(-ns // case["batch"])
        return dict(bytes=3.0 * ns * (247 + 6) * 4 + batches * par * 30.0, flops=ns * par * (6.0 + 6.0 + 2.0))
    if k == "batch":
        edge = 0.5 * (case["lo"] + case["hi"])
        cells = case["cases"] * edge ** 3
        steps = case["steps"]
        extra = -(-steps // case["sample"]) * case["cases"] * 247 * 4.0 + case["cases"] * steps * 19 * 8.0
    else:
        nx, ny, nz = ((case["n"], case["n"], case.get("nz", case["n"])) if k != "sediment"
                      else (case["nxy"], case["nxy"], case["nz"]))
        cells, steps = float(nx * ny * nz), case["steps"]
        extra = cells * (19 * ESZ[case.get("storage", "f32")] + 4 * (8 if case.get("storage") == "f64" else 4))
    per = 2 * 19 * ESZ[case.get("storage", "f32")] + 1
    return dict(bytes=cells * steps * per + extra, flops=cells * steps * 230.0)


# ------------------------------------------------------------------ the same in 64 bits, plain torch
_C = [(0, 0, 0)] + [(x, y, z) for x in (-1, 0, 1) for y in (-1, 0, 1) for z in (-1, 0, 1)
                    if 0 < abs(x) + abs(y) + abs(z) < 3]
_W = [1 / 3.0 if not any(c) else (1 / 18.0 if sum(map(abs, c)) == 1 else 1 / 36.0) for c in _C]
_OPP = [_C.index(tuple(-a for a in c)) for c in _C]


def _rot(q):
    w, x, y, z = q
    return np.array([[1 - 2 * (y * y + z * z), 2 * (x * y - w * z), 2 * (x * z + w * y)],
                     [2 * (x * y + w * z), 1 - 2 * (x * x + z * z), 2 * (y * z - w * x)],
                     [2 * (x * z - w * y), 2 * (y * z + w * x), 1 - 2 * (x * x + y * y)]])


class _Lattice:
    """Two-lattice D3Q19 TRT with bounce-back on rigid fibers, FP64."""

    def __init__(self, shape, args, fibers, net=None):
        self.n = shape
        nx, ny, nz = shape
        self.dev = "cuda" if torch.cuda.is_available() else "cpu"
        self.wall = [2 if args.get("x_walls") == "free-slip" else 0, 2 if args.get("y_walls") == "free-slip" else 0,
                     0 if args.get("z_periodic") else (2 if args.get("z_free_slip") else 1)]
        self.per = [True, True, bool(args.get("z_periodic"))]
        self.U, self.tau, self.stab = args.get("wall_u", 0.0), args["tau"], args.get("stabilize", False)
        self.we, self.wo = 1.0 / self.tau, 1.0 / (0.5 + 3.0 / 16.0 / (self.tau - 0.5))
        self.net, self.gamma = net, 2.0 * args.get("wall_u", 0.0) / nz
        z = torch.arange(nz, dtype=torch.float64, device=self.dev)
        ux = self.U * (2.0 * (z + 0.5) / nz - 1.0) if args.get("init_couette") else torch.zeros_like(z)
        self.f = torch.empty((19, nz, ny, nx), dtype=torch.float64, device=self.dev)
        for q in range(19):
            cu = _C[q][0] * ux
            self.f[q] = (_W[q] * (3 * cu + 4.5 * cu * cu - 1.5 * ux * ux))[:, None, None]
        self.owner = torch.full((nz, ny, nx), -1, dtype=torch.int64, device=self.dev)
        self.fib = []
        for f in fibers:
            L, r = f["length"], f["radius"]
            sph = f.get("shape") == "spherocylinder"
            rho = f.get("density_ratio", 1.0)
            h = L - 2 * r if sph else L
            mc, ms = rho * math.pi * r * r * h, rho * 4 / 3 * math.pi * r ** 3 if sph else 0.0
            ipar = 0.5 * mc * r * r + 0.4 * ms * r * r
            iper = mc * (3 * r * r + h * h) / 12 + ms * (0.4 * r * r + 0.25 * h * h + 0.375 * h * r)
            q = np.asarray(f["q"], float)
            b = dict(L=L, r=r, sph=sph, m=mc + ms, ipar=ipar, iper=iper, X=np.array(f["X"], float),
                     q=q / np.linalg.norm(q), V=np.array(f.get("V", (0, 0, 0)), float),
                     W=np.array(f.get("W", (0, 0, 0)), float), fe=np.array(f.get("force", (0, 0, 0)), float), prev=None)
            b["t"] = _rot(b["q"])[:, 0]
            b["Lam"] = iper * b["W"] + (ipar - iper) * (b["t"] @ b["W"]) * b["t"]
            self.fib.append(b)
        self._map()

    def _rel(self, p, X):
        """Minimum-image vectors from X to the cells p [N][3]."""
        d = p - torch.as_tensor(X, dtype=torch.float64, device=self.dev)
        for k in range(3):
            if self.per[k]:
                n = float(self.n[k])
                d[:, k] = torch.where(d[:, k] > n / 2, d[:, k] - n, torch.where(d[:, k] < -n / 2, d[:, k] + n, d[:, k]))
        return d

    def _motion(self, p, own, name=("X", "V", "W")):
        """Lever arms and surface velocities at the cells p of the fibers own."""
        X, V, W = (torch.tensor(np.array([b[k] for b in self.fib]), device=self.dev)[own] for k in name)
        r = self._rel(p, X)
        return r, V + torch.cross(W, r, dim=1)

    def _map(self):
        self.owner.fill_(-1)
        for i in range(len(self.fib) - 1, -1, -1):      # the lowest index keeps an overlapped cell
            b = self.fib[i]
            ax = []
            for k in range(3):
                e = (0.5 * b["L"]) * abs(b["t"][k]) + b["r"] + 1.0
                lo, hi = math.floor(b["X"][k] - e), math.ceil(b["X"][k] + e)
                if not self.per[k]:
                    lo, hi = max(lo, 0), min(hi, self.n[k] - 1)
                ax.append(torch.arange(lo, hi + 1, device=self.dev) % self.n[k])
            p = torch.cartesian_prod(*ax)
            d = self._rel(p.double(), b["X"])
            t = torch.tensor(b["t"], device=self.dev)
            a = d @ t
            q, hl, r2 = (d * d).sum(1) - a * a, 0.5 * b["L"], b["r"] ** 2
            if b["sph"]:
                e = (a.abs() - (hl - b["r"])).clamp(min=0.0)
                ok = q + e * e <= r2
            else:
                ok = (a * a <= hl * hl) & (q <= r2)
            p = p[ok]
            self.owner[p[:, 2], p[:, 1], p[:, 0]] = i

    def _momentum(self):
        j = [torch.zeros_like(self.f[0]) for _ in range(3)]
        for q in range(1, 19):
            for k in range(3):
                if _C[q][k]:
                    j[k].add_(self.f[q], alpha=float(_C[q][k]))
        return j

    def fields(self):
        rho, u = 1.0 + self.f.sum(0), torch.stack(self._momentum())
        s = (self.owner >= 0).nonzero()
        if len(s):
            z, y, x = s.T
            rho[z, y, x] = 1.0
            u[:, z, y, x] = self._motion(s.flip(1).double(), self.owner[z, y, x])[1].T
        return rho, u

    def _pull(self, q):
        """Populations streaming into every cell along c_q (walls, no fibers)."""
        c = _C[q]
        sh = [(2 - k, c[k]) for k in range(3) if c[k]]
        out = torch.roll(self.f[q], [s for _, s in sh], [d for d, _ in sh]) if sh else self.f[q].clone()
        dims = [k for k in range(3) if c[k] and self.wall[k]]
        for m in range(1, 1 << len(dims)):
            cross = [dims[i] for i in range(len(dims)) if m >> i & 1]
            dst = [slice(None)] * 3
            for k in dims:
                lo, hi = (0, 1) if c[k] > 0 else (self.n[k] - 1, self.n[k])
                dst[2 - k] = slice(lo, hi) if k in cross else (slice(1, None) if c[k] > 0 else slice(0, -1))
            if any(self.wall[k] == 1 for k in cross):
                v = self.f[_OPP[q]][tuple(dst)]
                if 2 in cross and self.wall[2] == 1:
                    v = v + 6 * _W[q] * c[0] * (-self.U if c[2] > 0 else self.U)
                out[tuple(dst)] = v
            else:
                rq = _C.index(tuple(-c[k] if k in cross else c[k] for k in range(3)))
                src = [dst[2 - k] if k in cross else slice(None) for k in (2, 1, 0)]
                v = self.f[rq][tuple(src)]
                rest = [k for k in range(3) if c[k] and k not in cross]
                if rest:
                    v = torch.roll(v, [c[k] for k in rest], [2 - k for k in rest])
                keep = [slice(None) if k in cross else dst[2 - k] for k in (2, 1, 0)]
                out[tuple(dst)] = v[tuple(keep)]
        return out

    def step(self):
        corr = self._closure() if self.net is not None else None
        j = self._momentum()
        drho = self.f.sum(0)
        ub = [0.0] * 3
        if self.stab:
            fl = self.owner < 0
            ub = [float(j[k][fl].mean()) for k in range(3)]
        u = [j[k] - ub[k] for k in range(3)]
        del j
        base = drho - 1.5 * (u[0] ** 2 + u[1] ** 2 + u[2] ** 2)
        f = self.f
        f[0] -= self.we * (f[0] - _W[0] * base)
        for q in range(1, 19):
            o = _OPP[q]
            if o < q:
                continue
            cu = sum(c * v for c, v in zip(_C[q], u) if c)
            de = self.we * (0.5 * (f[q] + f[o]) - _W[q] * (base + 4.5 * cu * cu))
            dd = self.wo * (0.5 * (f[q] - f[o]) - 3 * _W[q] * cu)
            f[q] -= de + dd
            f[o] -= de - dd
        del base, drho, u
        new = torch.empty_like(f)
        for q in range(19):
            new[q] = self._pull(q)
        np_ = len(self.fib)
        s = (self.owner >= 0).nonzero()
        if len(s):
            ys = s.flip(1)
            oy = self.owner[s[:, 0], s[:, 1], s[:, 2]]
            F0, M0 = (torch.zeros((np_, 3), dtype=torch.float64, device=self.dev) for _ in range(2))
            A, B, Cm = (torch.zeros((np_, 3, 3), dtype=torch.float64, device=self.dev) for _ in range(3))
            for q in range(1, 19):
                c = torch.tensor(_C[q], device=self.dev)
                x = ys + c
                ok = torch.ones(len(x), dtype=torch.bool, device=self.dev)
                for k in range(3):
                    if self.per[k]:
                        x[:, k] %= self.n[k]
                    else:
                        ok &= (x[:, k] >= 0) & (x[:, k] < self.n[k])
                x, y, o = x[ok], ys[ok], oy[ok]
                ok = self.owner[x[:, 2], x[:, 1], x[:, 0]] < 0
                x, y, o = x[ok], y[ok], o[ok]
                if not len(x):
                    continue
                d = (-c).double()                       # from the fluid cell x to the solid cell y
                ft = f[_OPP[q], x[:, 2], x[:, 1], x[:, 0]]
                r, us = self._motion(y.double(), o)
                new[q, x[:, 2], x[:, 1], x[:, 0]] = ft - 6 * _W[q] * (us @ d)
                dF = (2 * (ft + _W[q]))[:, None] * d
                rc = torch.cross(r, d.expand_as(r), dim=1)
                cc = d.expand_as(r)
                F0.index_add_(0, o, dF)
                M0.index_add_(0, o, torch.cross(r, dF, dim=1))
                k6 = 6 * _W[q]
                A.index_add_(0, o, k6 * cc[:, :, None] * cc[:, None, :])
                B.index_add_(0, o, k6 * cc[:, :, None] * rc[:, None, :])
                Cm.index_add_(0, o, k6 * rc[:, :, None] * rc[:, None, :])
            F0, M0, A, B, Cm = (v.cpu().numpy() for v in (F0, M0, A, B, Cm))
        self.f = new
        del f
        rows = []
        for i, b in enumerate(self.fib):
            F0u, M0u = (F0[i], M0[i]) if b["prev"] is None else (0.5 * (F0[i] + b["prev"][0]), 0.5 * (M0[i] + b["prev"][1]))
            if corr is not None:
                F0u, M0u = F0u + corr[i, :3], M0u + corr[i, 3:]
            Iw = b["iper"] * np.eye(3) + (b["ipar"] - b["iper"]) * np.outer(b["t"], b["t"])
            K = np.block([[b["m"] * np.eye(3) + A[i], B[i]], [B[i].T, Iw + Cm[i]]])
            v = np.linalg.solve(K, np.concatenate([b["m"] * b["V"] + F0u + b["fe"], b["Lam"] + M0u]))
            F, M = F0u - A[i] @ v[:3] - B[i] @ v[3:], M0u - B[i].T @ v[:3] - Cm[i] @ v[3:]
            for k in ("X", "V", "W"):
                b[k + "0"] = b[k]
            b["prev"], b["V"], b["W"], b["Lam"] = (F0[i], M0[i]), v[:3], v[3:], b["Lam"] + M
            X = b["X"] + b["V"]
            b["X"] = np.array([X[k] % self.n[k] if self.per[k] else X[k] for k in range(3)])
            a = np.linalg.norm(b["W"])
            d = np.concatenate([[math.cos(a / 2)], (math.sin(a / 2) / a if a else 0.0) * b["W"]])
            p = b["q"]
            q = np.concatenate([[d[0] * p[0] - d[1:] @ p[1:]], d[0] * p[1:] + p[0] * d[1:] + np.cross(d[1:], p[1:])])
            b["q"] = q / np.linalg.norm(q)
            b["t"] = _rot(b["q"])[:, 0]
            rows.append(np.concatenate([F, M, b["X"], b["q"], b["V"], b["W"]]))
        if len(s):
            old = self.owner.clone()
            self._map()
            bare = ((old >= 0) & (self.owner < 0)).nonzero()
            if len(bare):
                z, y, x = bare.T
                us = self._motion(bare.flip(1).double(), old[z, y, x], ("X0", "V0", "W0"))[1]
                uu = (us * us).sum(1)
                for q in range(19):
                    cu = us @ torch.tensor(_C[q], dtype=torch.float64, device=self.dev)
                    self.f[q, z, y, x] = _W[q] * (3 * cu + 4.5 * cu * cu - 1.5 * uu)
        return np.array(rows)

    def features(self):
        """[np][247]: trilinear velocities relative to the rigid motion on the
        3 x 27 stencil in the body frame over gamma L, and the quaternion."""
        u = self.fields()[1].cpu().numpy()
        nx, ny, nz = self.n
        out = np.zeros((len(self.fib), 247))
        m = np.arange(27)
        ob = 2.0 * np.stack([m % 3 - 1, m // 3 % 3 - 1, m // 9 - 1], 1)
        for i, b in enumerate(self.fib):
            R = _rot(b["q"])
            d = np.concatenate([side * R[:, 0] + ob @ R.T for side in (0.0, 0.5 * b["L"], -0.5 * b["L"])])
            p = b["X"] + d
            p[:, 2] = np.clip(p[:, 2], 0.0, nz - 1.0)
            i0 = np.floor(p).astype(int)
            i0[:, 2] = np.minimum(i0[:, 2], nz - 2)
            a = p - i0
            val = np.zeros((81, 3))
            for c in range(8):
                s = np.array([c & 1, c >> 1 & 1, c >> 2])
                w = np.prod(np.where(s, a, 1 - a), axis=1)
                x, y, z = (i0 + s).T
                val += w[:, None] * u[:, z, y % ny, x % nx].T
            rel = (val - b["V"] - np.cross(b["W"], d)) @ R / (self.gamma * b["L"])
            out[i] = np.concatenate([rel.ravel(), -b["q"] if b["q"][0] < 0 else b["q"]])
        return out

    def _closure(self):
        x, nu = self.features(), (self.tau - 0.5) / 3.0
        n = self.net
        y = _mlp(_bf16(n["params"]), (x - n["in_mean"]) * n["in_inv_std"])[0] * n["out_scale"]
        y[~np.all((x >= n["env_min"]) & (x <= n["env_max"]), axis=1)] = 0.0
        out = np.zeros((len(self.fib), 6))
        for i, b in enumerate(self.fib):
            R, s = _rot(b["q"]), nu * self.gamma * b["L"] ** 2
            out[i] = np.concatenate([R @ y[i, :3] * s, R @ y[i, 3:] * s * b["L"]])
        return out


def _bf16(w):
    return torch.tensor(w, dtype=torch.float32).bfloat16().double().numpy()


def _mlp(w, x, t=None):
    """Network outputs in FP64; with targets also the mean squared error and its gradient."""
    w, x = torch.tensor(w, dtype=torch.float64), torch.tensor(np.asarray(x, np.float64))
    w.requires_grad_(t is not None)
    a = torch.split(w, [64 * 247, 64, 64 * 64, 64, 6 * 64, 6])
    h = torch.nn.functional.gelu(x @ a[0].view(64, 247).T + a[1])
    h = torch.nn.functional.gelu(h @ a[2].view(64, 64).T + a[3])
    y = h @ a[4].view(6, 64).T + a[5]
    if t is None:
        return y.numpy(), None, None
    loss = ((y - torch.tensor(np.asarray(t, np.float64))) ** 2).mean()
    loss.backward()
    return y.detach().numpy(), float(loss.detach()), w.grad.numpy()


def _exact_sbf(case, sc):
    dev = "cuda" if torch.cuda.is_available() else "cpu"
    T = lambda a: torch.tensor(np.asarray(a), dtype=torch.float64, device=dev)  # noqa: E731
    X, p, F = T(sc.X), T(sc.p), T(sc.F)
    m, N, l, L = len(sc.X), case["modes"], 0.5 * sc.length, sc.length
    r, d = sc.eps * L, -math.log(sc.eps ** 2 * math.e)
    g, gw = np.polynomial.legendre.leggauss(3)
    h = 2.0 / case["nq"]
    t = np.concatenate([-1 + h * (i + 0.5) + 0.5 * h * g for i in range(case["nq"])])
    wt = np.concatenate([0.5 * h * gw * l] * case["nq"])
    P = np.stack([np.polynomial.legendre.legval(t, np.eye(N + 1)[n]) for n in range(N + 1)])
    s, A = T(l * t), T(P * wt)
    Ln = [0.0] + [-2.0 * sum(1.0 / i for i in range(1, n + 1)) for n in range(1, N + 1)]
    cn = T((2.0 * np.arange(N + 1) + 1) / (2 * l))
    eye = torch.eye(3, dtype=torch.float64, device=dev)
    prev, part = None, max(1, 2048 // m)
    for _ in range(case["steps"]):
        th = torch.zeros((m, N + 1, 3, m, N + 1, 3), dtype=torch.float64, device=dev)
        for a in range(0, m, part):
            e = min(m, a + part)
            R = ((X[a:e, None] - X[None])[:, :, None, None] + s[:, None, None] * p[a:e, None, None, None]
                 - s[:, None] * p[None, :, None, None])
            n2 = (R * R).sum(-1)
            n2[torch.arange(e - a), torch.arange(a, e)] = 1.0
            i1 = n2.rsqrt()
            al, be = i1 + 0.5 * r * r * i1 ** 3, i1 ** 3 - 1.5 * r * r * i1 ** 5
            for x in range(3):
                for y in range(x, 3):
                    v = torch.matmul(torch.matmul(A, be * R[..., x] * R[..., y] + (al if x == y else 0.0)), A.T)
                    v[torch.arange(e - a), torch.arange(a, e)] = 0.0
                    th[a:e, :, x, :, :, y] = v.transpose(1, 2)
                    th[a:e, :, y, :, :, x] = v.transpose(1, 2)
        pp = p[:, :, None] * p[:, None, :]
        lam = d * (eye + pp) + 2 * (eye - pp)
        known = torch.einsum("mnayb,yb->mna", th[:, :, :, :, 0, :], F / (2 * l))
        S = th[:, 1:, :, :, 1:, :] * cn[1:, None, None, None, None]
        rhs = -known[:, 1:] * cn[1:, None]
        S[:, 0] = torch.einsum("mab,mbykc->maykc", pp, S[:, 0])
        rhs[:, 0] = torch.einsum("mab,mb->ma", pp, rhs[:, 0])       # no torque in these cases
        i = torch.arange(m, device=dev)
        for n in range(1, N + 1):
            own = lam + Ln[n] * (eye + pp)
            if n == 1:
                own = (eye - pp) + torch.matmul(pp, own)
            S[i, n - 1, :, i, n - 1, :] += own
        a = torch.linalg.solve(S.reshape(3 * m * N, 3 * m * N), rhs.reshape(-1)).view(m, N, 3)
        I = known[:, :2] + torch.matmul(th[:, :2, :, :, 1:].reshape(m * 6, 3 * m * N), a.reshape(-1)).view(m, 2, 3)
        V = (torch.matmul(lam, F[:, :, None])[..., 0] + I[:, 0]) / (8 * math.pi * L)
        W = 3.0 / (2 * math.pi * L ** 3) * l * (I[:, 1] - p * (p * I[:, 1]).sum(1, keepdim=True))
        dV, dW = (V, W) if prev is None else (1.5 * V - 0.5 * prev[0], 1.5 * W - 0.5 * prev[1])
        X, p, prev = X + case["dt"] * dV, p + case["dt"] * dW, (V, W)
        p = p / p.norm(dim=1, keepdim=True)
    return {k: v.cpu().numpy() for k, v in dict(X=X, p=p, V=V, W=W).items()}


def exact(case, seed):
    k = case["kind"]
    if k == "sbf":
        return _exact_sbf(case, _sbf_scene(case, seed)) if case["m"] <= 400 else None
    if k == "fit":
        # an epoch of Adam updates grows rounding differences: no exact weights
        X, T, norm, w = _fit_data(case, seed)
        xn = (X.astype(np.float64) - norm.in_mean) * norm.in_inv_std
        _, loss, grad = _mlp(_bf16(w), xn, T)
        return {"loss": loss, "grad": grad, "losses": None, "weights": None, "y": None}
    if k == "batch":
        if case["cases"] * case["steps"] > 1200:
            return None
        feats, hist = [], []
        for sc in _batch_cases(case, seed):
            fb = sc.fibers[0]
            g = _Lattice((sc.nx, sc.ny, sc.nz), dict(tau=sc.tau, wall_u=sc.wall_u, init_couette=True),
                         [dict(X=fb.X, q=fb.q, length=fb.length, radius=fb.radius, V=fb.V, W=fb.W)])
            fe, h = [], []
            for i in range(case["steps"]):
                if i % case["sample"] == 0:
                    fe.append(g.features()[0])
                h.append(g.step()[0])
            feats.append(fe)
            hist.append(h)
        return {"features": np.array(feats).transpose(1, 0, 2), "history": np.array(hist)}
    shape, args, fibers = _scene(case, seed)
    cost = case["steps"] * (shape[0] * shape[1] * shape[2] / 4e6 + 0.6 * len(fibers) + 4.0)
    if cost > 5500:
        return None
    net = dict(np.load(NET)) if case.get("closure") else None
    g = _Lattice(shape, args, fibers, net)
    hist = np.array([g.step() for _ in range(case["steps"])])
    rho, u = g.fields()
    return {"history": hist, "rho": rho, "u": u}
