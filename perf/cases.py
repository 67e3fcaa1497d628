"""Timed cases of the solver: what a user's program calls, over the sizes that it meets.

Eight kinds of work, each through the package's public entry points:

* "solve": one (F)GMRES solve on a context that the program keeps (many sources on one medium);
* "medium": everything that a new medium costs: set-up, right-hand side, solve, release (training data generation);
* "direct": one application of the preconditioner as the direct solver of the second-order system;
* "operator": the compact right-hand side and one product y = A x;
* "waves": one batch of plane-wave sources on one medium;
* "uneven": one batch of media of different sizes;
* "infer": a learned initial guess: features, network, prolongation to the solver's grid;
* "train": one training step of that network.

All inputs are made on the GPU from the seed. exact() gives the same results in 64 bits with plain torch: dense 1D
eigenvectors, shifted-array stencils, full GMRES, and convolutions as sums over taps.
"""
import math

import numpy as np
import torch

import paper_2602_07711_amd as H

DEV = "cuda"
C128 = torch.complex128
KINDS = ("solve", "medium", "direct", "operator", "waves", "uneven", "infer", "train")


def listed():
    return [
        # the smallest solve: 32^3, constant medium, 4th order, a handful of iterations; launches and the host's share count
        dict(name="solve_gauss32", kind="solve", medium="constant", nx=32, ny=32, nz=32, order=4, k0=20.0, prec="eigt",
             fp32=False, m=30),
        # generating one training sample of the learned warm start: a new 64^3 medium is set up, solved once, released
        dict(name="medium_inclusions64", kind="medium", medium="inclusions", nx=64, ny=64, nz=64, order=6, k0=30.0,
             prec="eigt", fp32=True, m=50),
        # the ordinary solve: 128^3, four smooth inclusions, FP32 preconditioner
        dict(name="solve_inclusions128", kind="solve", medium="inclusions", nx=128, ny=128, nz=128, order=6, k0=60.0,
             prec="eigt", fp32=True, m=50),
        # the benchmark's workload: 256^3 filtered noise, FP32 preconditioner
        dict(name="solve_noise256", kind="solve", medium="noise", nx=256, ny=256, nz=256, order=6, k0=120.0,
             prec="eigt", fp32=True, m=50),
        # the paper's scattering problem (attenuating inclusion, odd size), all in FP64, with the sine-transform path
        dict(name="solve_scatter127", kind="solve", medium="sphere", nx=127, ny=127, nz=127, order=6,
             k0=math.sqrt(439.2), prec="pfft", fp32=False, m=50),
        # the paper's direct solves of the second-order system: 200^3 (no multiple of a tile) and 255^3 (odd)
        dict(name="direct_eigt200", kind="direct", nx=200, ny=200, nz=200, k0=math.sqrt(439.2), prec="eigt"),
        dict(name="direct_pfft255", kind="direct", nx=255, ny=255, nz=255, k0=math.sqrt(439.2), prec="pfft"),
        # residual checks and new sources on a box that is no cube and no multiple of anything
        dict(name="operator_box", kind="operator", nx=250, ny=190, nz=217, order=6, k0=90.0),
        # many incident directions on one medium, and a set of different problems, each as one batch
        dict(name="batch_waves128", kind="waves", n=128, count=16, k0=60.0, fp32=True, m=30),
        dict(name="batch_uneven", kind="uneven", n_lo=64, n_hi=128, count=8, fp32=True, m=30),
        # the learned warm start: inference for a 128^3 problem and one training step, at the size it is trained at
        dict(name="infer64", kind="infer", size=64, nf=128, bf16=True),
        dict(name="train64", kind="train", size=64, batch=4, bf16=True),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(KINDS)
    if kind in ("solve", "medium"):
        n = _log_int(rng, 24, 208 if kind == "solve" else 112)
        prec = rng.choice(("eigt", "eigt", "pfft"))
        order = rng.choice((4, 6, 6))
        # boxes have another extent along each axis (the 6th order keeps h the same on all)
        dims = [n, n, n] if rng.random() < 0.5 else [max(20, int(n * rng.uniform(0.6, 1.0))) for _ in range(3)]
        return dict(kind=kind, medium=rng.choice(("inclusions", "noise")), nx=dims[0], ny=dims[1], nz=dims[2],
                    order=order, k0=round(min(60.0, 0.465 * (max(dims) + 1)) * rng.uniform(0.5, 1.0), 3), prec=prec,
                    fp32=rng.random() < 0.6, m=rng.choice((30, 50)))
    if kind == "direct":
        d = [_log_int(rng, 40, 255) for _ in range(3)] if rng.random() < 0.5 else [_log_int(rng, 40, 255)] * 3
        return dict(kind=kind, nx=d[0], ny=d[1], nz=d[2], k0=round(rng.uniform(10.0, 40.0), 3),
                    prec=rng.choice(("eigt", "pfft")))
    if kind == "operator":
        d = [_log_int(rng, 24, 240) for _ in range(3)]
        return dict(kind=kind, nx=d[0], ny=d[1], nz=d[2], order=rng.choice((4, 6)),
                    k0=round(0.4 * (max(d) + 1) * rng.uniform(0.5, 1.0), 3))
    if kind == "waves":
        return dict(kind=kind, n=_log_int(rng, 40, 112), count=rng.randint(2, 16), k0=round(rng.uniform(15.0, 45.0), 3),
                    fp32=rng.random() < 0.75, m=30)
    if kind == "uneven":
        lo = _log_int(rng, 32, 72)
        return dict(kind=kind, n_lo=lo, n_hi=int(lo * rng.uniform(1.2, 1.75)), count=rng.randint(2, 8),
                    fp32=rng.random() < 0.75, m=30)
    size = 8 * rng.randint(3, 8)
    if kind == "infer":
        return dict(kind=kind, size=size, nf=rng.randint(size, 2 * size + 1), bf16=rng.random() < 0.75)
    return dict(kind=kind, size=size, batch=rng.randint(1, 4), bf16=rng.random() < 0.75)


# ------------------------------------------------------------------------------------------------ inputs

RTOL = 1e-10


def _rng(seed):
    return np.random.default_rng(seed)


def _axes(n3, h, shift=0.0):
    """Node coordinates with the two-cell halo, (z, y, x) broadcastable; the unit cube's nodes i h for a cube."""
    out = []
    for a, n in enumerate(n3):
        c = (torch.arange(n + 4, dtype=torch.float64, device=DEV) - 1 - shift) * h
        out.append(c.reshape([-1 if b == a else 1 for b in range(3)]))
    return out


def _noise(shape, seed, sigma=8):
    """Uniform noise under a separable Gaussian of `sigma` cells, normalised to max |w| = 1."""
    g = torch.Generator(device=DEV).manual_seed(int(seed))
    r = 4 * sigma
    w = torch.rand([s + 2 * r for s in shape], generator=g, dtype=torch.float64, device=DEV) * 2 - 1
    t = torch.arange(-r, r + 1, dtype=torch.float64)
    k = torch.exp(-t * t / (2.0 * sigma * sigma))
    k = (k / k.sum()).tolist()
    for a in range(3):
        out = torch.zeros_like(w.narrow(a, 0, shape[a]))
        for i, v in enumerate(k):
            out.add_(w.narrow(a, i, shape[a]), alpha=v)
        w = out
    return w / w.abs().max()


def _medium(kind, n3, h, k0, seed):
    """k^2 with its two-cell halo, (z, y, x)."""
    shape = [n + 4 for n in n3]
    if kind == "constant":
        return torch.full(shape, k0 * k0, dtype=torch.float64, device=DEV)
    if kind == "noise":
        return k0 * k0 * (1.0 + 0.2 * _noise(shape, seed))
    z, y, x = _axes(n3, h, 0.5 if kind == "sphere" else 0.0)
    r = _rng(seed)
    size = [h * (n + 1) for n in n3]
    if kind == "sphere":
        c = 0.5 + r.uniform(-0.2, 0.2, size=3)
        inside = (z - c[0]) ** 2 + (y - c[1]) ** 2 + (x - c[2]) ** 2 <= 0.01
        return torch.where(inside, torch.tensor(1050 + 2.26j, dtype=C128, device=DEV),
                           torch.tensor(k0 * k0 + 0j, dtype=C128, device=DEV)).contiguous()
    b = torch.zeros(shape, dtype=torch.float64, device=DEV)
    for c in r.uniform(0.2, 0.8, size=(4, 3)):
        b += torch.exp(-((z - c[0] * size[0]) ** 2 + (y - c[1] * size[1]) ** 2 + (x - c[2] * size[2]) ** 2) / 0.02)
    return k0 * k0 * (1.0 + 0.3 * b)


def _gauss(n3, h, seed, width=2.0):
    """A Gaussian source of `width` cells near the middle."""
    z, y, x = _axes(n3, h)
    c = [h * (n + 1) * v for n, v in zip(n3, _rng((seed, 77)).uniform(0.35, 0.65, size=3))]
    r2 = (z - c[0]) ** 2 + (y - c[1]) ** 2 + (x - c[2]) ** 2
    return torch.exp(-r2 / (2 * (width * h) ** 2)).to(C128).contiguous()


def _wave(k2, k0, n3, h, d, shift=0.0):
    """Scattering source of the incident plane wave exp(i k0 d . x)."""
    z, y, x = _axes(n3, h, shift)
    ph = k0 * (d[0] * x + d[1] * y + d[2] * z)
    return (-(k2 - k0 * k0) * torch.polar(torch.ones_like(ph), ph)).contiguous()


def _problem(case, seed):
    n3 = (case["nz"], case["ny"], case["nx"])
    sphere = case["medium"] == "sphere"
    h = 1.0 / max(n3) if sphere else 1.0 / (max(n3) + 1)
    k2 = _medium(case["medium"], n3, h, case["k0"], seed)
    f = _wave(k2, case["k0"], n3, h, _dirs(1, seed)[0], 0.5) if sphere else _gauss(n3, h, seed)
    return n3, h, k2, f


def _dirs(count, seed):
    g = _rng((seed, 4)).standard_normal((count, 3))
    return g / np.linalg.norm(g, axis=1, keepdims=True)


def _wavy(n3, k0h, seed):
    """A field like a solution: plane waves of the background plus small noise, complex128, flat."""
    g = torch.Generator(device=DEV).manual_seed(int(seed))
    z, y, x = (a.squeeze() for a in _axes(n3, 1.0))
    z, y, x = z[2:-2, None, None], y[None, 2:-2, None], x[None, None, 2:-2]
    u = 0.01 * torch.randn(n3, generator=g, dtype=C128, device=DEV)
    for d in _dirs(4, seed):
        ph = k0h * (d[0] * x + d[1] * y + d[2] * z)
        u += torch.polar(torch.ones_like(ph), ph)
    return u.reshape(-1).contiguous()


def _uneven(case, seed):
    c = case["count"]
    ks = _rng((seed, 40)).uniform(0.25, 0.465, size=c)
    ns = [int(round(case["n_lo"] + (case["n_hi"] - case["n_lo"]) * p / (c - 1))) for p in range(c)]
    return [(n, min(60.0, float(k) * (n + 1))) for n, k in zip(ns, ks)]


# (inputs, outputs, taps, level) of the network's convolutions
CONVS = [(2, 16, 27, 0), (16, 16, 27, 0), (16, 32, 27, 1), (32, 32, 27, 1), (32, 64, 27, 2), (64, 64, 27, 2),
         (64, 64, 27, 3), (64, 64, 27, 3), (128, 64, 27, 2), (96, 32, 27, 1), (48, 16, 27, 0), (16, 2, 1, 0)]
NET_K0 = 60.0


def _weights(seed):
    """He-uniform weights and small biases, in the network's order."""
    r = _rng((seed, 5))
    out = []
    for ci, co, taps, _ in CONVS:
        a = math.sqrt(6.0 / (ci * taps))
        out += [r.uniform(-a, a, size=co * ci * taps), r.uniform(-0.05, 0.05, size=co)]
    return torch.from_numpy(np.concatenate(out).astype(np.float32))


def _net(case, seed):
    net = H.Cnn(case["size"], max_batch=case.get("batch", 1), bf16=case["bf16"])
    net.set_params(_weights(seed))
    return net


def _train_data(case, seed):
    """Contrast and source channels of one batch, and targets of unit RMS that look like fields."""
    S, B = case["size"], case["batch"]
    xs, ts = [], []
    for b in range(B):
        n3, h = (S, S, S), 1.0 / (S + 1)
        k2 = _medium("inclusions", n3, h, NET_K0, (seed, b))[2:-2, 2:-2, 2:-2]
        f = _gauss(n3, h, (seed, b), 0.03 / h)[2:-2, 2:-2, 2:-2].real
        xs.append(torch.stack([(k2 / NET_K0 ** 2 - 1).reshape(-1), f.reshape(-1)]))
        u = _wavy(n3, 0.46, _rng((seed, b, 9)).integers(1 << 30)) / 2
        ts.append(torch.stack([u.real, u.imag]))
    return torch.stack(xs).float().contiguous(), torch.stack(ts).float().contiguous()


def _infer_data(case, seed):
    nf = case["nf"]
    n3, h = (nf, nf, nf), 1.0 / (nf + 1)
    return _medium("inclusions", n3, h, NET_K0, seed).contiguous(), _gauss(n3, h, seed, 0.03 / h)


# ------------------------------------------------------------------------------------------------ the passes

def prepare(case, seed):
    kind = case["kind"]
    s = dict(case)
    if kind in ("solve", "medium"):
        n3, h, k2, f = _problem(case, seed)
        s.update(n3=n3, h=h)
        if kind == "solve":
            s["ctx"] = H.helm_setup(k2, h, case["order"], "abc", case["k0"])
            s["F"] = H.helm_rhs(s["ctx"], f)
        else:
            s.update(k2=k2, f=f)
    elif kind == "direct":
        n3 = (case["nz"], case["ny"], case["nx"])
        h = 1.0 / max(n3)
        k2 = _medium("constant", n3, h, case["k0"], seed)
        s["ctx"] = H.helm_setup(k2, h, 2, "abc", case["k0"])
        s["y"] = _wavy(n3, case["k0"] * h, seed)
    elif kind == "operator":
        n3 = (case["nz"], case["ny"], case["nx"])
        h = 1.0 / (max(n3) + 1)
        k2 = _medium("inclusions", n3, h, case["k0"], seed)
        s["ctx"] = H.helm_setup(k2, h, case["order"], "abc", case["k0"])
        s["f"] = _wave(k2, case["k0"], n3, h, _dirs(1, seed)[0])
        s["x"] = _wavy(n3, case["k0"] * h, seed)
    elif kind == "waves":
        n3, h = (case["n"],) * 3, 1.0 / (case["n"] + 1)
        k2 = _medium("inclusions", n3, h, case["k0"], seed)
        ctx = H.helm_setup(k2, h, 6, "abc", case["k0"])
        s["Fs"] = [H.helm_rhs(ctx, _wave(k2, case["k0"], n3, h, d)) for d in _dirs(case["count"], seed)]
        s["batch"] = H.helm_batch_create([ctx] * case["count"], m=case["m"], prec_fp32=case["fp32"])
    elif kind == "uneven":
        ctxs, s["Fs"] = [], []
        for p, (n, k0) in enumerate(_uneven(case, seed)):
            n3, h = (n, n, n), 1.0 / (n + 1)
            ctxs.append(H.helm_setup(_medium("inclusions", n3, h, k0, (seed, p)), h, 6, "abc", k0))
            s["Fs"].append(H.helm_rhs(ctxs[-1], _gauss(n3, h, (seed, p))))
        s["batch"] = H.helm_batch_create(ctxs, m=case["m"], prec_fp32=case["fp32"])
    elif kind == "infer":
        s["net"] = _net(case, seed)
        s["k2"], s["f"] = _infer_data(case, seed)
        s["x"] = torch.empty(1, 2, case["size"] ** 3, dtype=torch.float32, device=DEV)
        s["y"] = torch.empty_like(s["x"])
        s["x0"] = torch.empty(case["nf"] ** 3, dtype=C128, device=DEV)
    else:
        s["net"] = _net(case, seed)
        s["x"], s["t"] = _train_data(case, seed)
    return s


def _gamma(k0, h):
    return (2 + 1j * k0 * h) / (2 - 1j * k0 * h)


def run(s):
    kind = s["kind"]
    if kind == "solve":
        return H.helm_gmres_solve(s["ctx"], s["F"], m=s["m"], rtol=RTOL, flexible=s["fp32"], prec=s["prec"],
                                  prec_fp32=s["fp32"])[0]
    if kind == "medium":
        ctx = H.helm_setup(s["k2"], s["h"], s["order"], "abc", s["k0"])
        F = H.helm_rhs(ctx, s["f"])
        x, _ = H.helm_gmres_solve(ctx, F, m=s["m"], rtol=RTOL, flexible=s["fp32"], prec=s["prec"], prec_fp32=s["fp32"])
        H.helm_destroy(ctx)
        return x
    if kind == "direct":
        return H.helm_precond_apply(s["ctx"], s["y"], kind=s["prec"])
    if kind == "operator":
        return {"F": H.helm_rhs(s["ctx"], s["f"]), "y": H.helm_matvec(s["ctx"], s["x"])}
    if kind in ("waves", "uneven"):
        return H.helm_batch_solve(s["batch"], s["Fs"], rtol=RTOL)[0]
    if kind == "infer":
        net = s["net"]
        net.features(s["k2"].reshape(-1), s["f"].reshape(-1), NET_K0, out=s["x"])
        net.forward(s["x"], s["y"])
        net.prolong(s["y"][0], s["nf"], gamma=_gamma(NET_K0, 1.0 / (s["size"] + 1)), fine=s["x0"], cubic=True)
        return {"y": s["y"], "x0": s["x0"]}
    loss = s["net"].train_step(s["x"], s["t"], 1e-4)
    return {"loss": loss, "grads": s["net"].grads()}


# ------------------------------------------------------------------------------------------------ the least work

def _solve_work(n, nx, ny, its, order, zbytes):
    # per iteration: read v and write z, the stencil's v, z, k^2 and result, and two passes over the basis so far
    per = its * (16 + zbytes + 16 + zbytes + 8 + 16) + 16 * sum(2 * j + 5 for j in range(its))
    # two transforms each way per axis, folded by their symmetry: 4 n flops per value
    return {"bytes": float(n) * per, "flops": float(n) * its * (8 * (nx + ny) + (250 if order == 6 else 100))}


def _its(k0):
    return int(10 + k0 / 7.5)     # about what the preconditioned iteration takes to RTOL


def work(case):
    kind = case["kind"]
    if kind in ("solve", "medium"):
        n = case["nx"] * case["ny"] * case["nz"]
        return _solve_work(n, case["nx"], case["ny"], _its(case["k0"]), case["order"], 8 if case["fp32"] else 16)
    if kind == "direct":
        n = case["nx"] * case["ny"] * case["nz"]
        return {"bytes": 32.0 * n, "flops": (8.0 if case["prec"] == "eigt" else 4.0) * n * (case["nx"] + case["ny"])}
    if kind == "operator":
        n = case["nx"] * case["ny"] * case["nz"]
        return {"bytes": (40.0 + 40.0) * n, "flops": 400.0 * n}
    if kind in ("waves", "uneven"):
        probs = [(case["n"], case["k0"])] * case["count"] if kind == "waves" else \
            [(n, 0.36 * n) for n, _ in _uneven(case, 0)]
        w = [_solve_work(n ** 3, n, n, _its(k0), 6, 8 if case["fp32"] else 16) for n, k0 in probs]
        return {k: sum(v[k] for v in w) for k in ("bytes", "flops")}
    V = case["size"] ** 3
    params = sum(ci * co * t + co for ci, co, t, _ in CONVS)
    fwd = sum(2.0 * ci * co * t * (case["size"] >> lv) ** 3 for ci, co, t, lv in CONVS)
    if kind == "infer":
        return {"bytes": 24.0 * (case["nf"] + 4) ** 3 + 16.0 * V + 16.0 * case["nf"] ** 3 + 4.0 * params, "flops": fwd}
    # input, target, parameters, both moments and the gradient; every activation written once and read once
    acts = sum(co * (case["size"] >> lv) ** 3 for _, co, _, lv in CONVS)
    return {"bytes": case["batch"] * (16.0 * V + 8.0 * acts) + 28.0 * params,
            "flops": case["batch"] * (3.0 * fwd - 2.0 * 2 * 16 * 27 * V)}


# ------------------------------------------------------------------------------------------------ 64 bits

def _ghost(u, g3):
    """One ghost layer per side, U_0 = gamma U_1 along each axis (z, y, x)."""
    for a in range(3):
        n = u.shape[a]
        u = torch.cat([g3[a] * u.narrow(a, 0, 1), u, g3[a] * u.narrow(a, n - 1, 1)], a)
    return u


def _at(u, o, pad):
    """The values at offset o = (dz, dy, dx) of an array with `pad` cells per side."""
    return u[tuple(slice(pad + d, u.shape[a] - pad + d) for a, d in enumerate(o))]


def _off(a, s=1):
    return tuple(s if b == a else 0 for b in range(3))


def _second(u, a):
    """The undivided second difference along one axis, one cell less per side there."""
    n = u.shape[a]
    return u.narrow(a, 0, n - 2) - 2 * u.narrow(a, 1, n - 2) + u.narrow(a, 2, n - 2)


def _inner(u, axes, by=1):
    for a in axes:
        u = u.narrow(a, by, u.shape[a] - 2 * by)
    return u


class _Exact:
    """A x and R f of the compact schemes on a uniform grid, and M^{-1}, in complex128."""

    def __init__(self, k2, n3, h, order, k0):
        self.n3, self.h, self.order = n3, h, order
        self.g3 = [_gamma(k0, h)] * 3
        self.k2h, self.k2 = k2, k2[2:-2, 2:-2, 2:-2]
        if order == 6:
            d = [(8 * (_at(k2, _off(a), 2) - _at(k2, _off(a, -1), 2)) - _at(k2, _off(a, 2), 2) + _at(k2, _off(a, -2), 2))
                 / (12 * h) for a in range(3)]
            lap = sum((16 * (_at(k2, _off(a), 2) + _at(k2, _off(a, -1), 2)) - 30 * self.k2 - _at(k2, _off(a, 2), 2)
                       - _at(k2, _off(a, -2), 2)) / (12 * h * h) for a in range(3))
            self.dk, self.lap = d, lap
        ev = {}
        for n in set(n3):
            T = -2 * np.eye(n, dtype=complex) + np.eye(n, k=1) + np.eye(n, k=-1)
            T[0, 0] += self.g3[0]
            T[-1, -1] += self.g3[0]
            w, V = np.linalg.eig(T)
            ev[n] = [torch.from_numpy(np.ascontiguousarray(v)).to(DEV) for v in (w, V, np.linalg.inv(V))]
        self.ev = [ev[n] for n in n3]
        wz, wy, wx = (e[0] for e in self.ev)
        self.sym = (wz[:, None, None] + wy[None, :, None] + wx[None, None, :]) / (h * h) + k0 * k0

    def precond(self, y):
        def along(mats, u):
            z, yy, x = self.n3
            u = torch.matmul(u.reshape(z * yy, x), mats[2].t().contiguous()).reshape(z, yy, x)
            u = torch.matmul(mats[0], u.reshape(z, yy * x)).reshape(z, yy, x)
            u = u.transpose(0, 1).reshape(yy, z * x)
            return torch.matmul(mats[1], u).reshape(yy, z, x).transpose(0, 1).contiguous()
        u = along([e[2] for e in self.ev], y.reshape(self.n3)) / self.sym
        return along([e[1] for e in self.ev], u).reshape(-1)

    def _mixed(self, u):
        """Sum over the axis pairs of the undivided products of second differences."""
        out = 0
        for a, b in ((0, 1), (0, 2), (1, 2)):
            out = out + _inner(_second(_second(u, a), b), [3 - a - b])
        return out

    def _lap(self, u):
        return sum(_inner(_second(u, a), [b for b in range(3) if b != a]) for a in range(3))

    def matvec(self, x):
        h, h2 = self.h, self.h ** 2
        u0 = x.reshape(self.n3)
        u, w = _ghost(u0, self.g3), _ghost(self.k2 * u0, self.g3)
        if self.order == 2:
            return (self._lap(u) / h2 + self.k2 * u0).reshape(-1)
        if self.order == 4:
            return (self._lap(u) / h2 + self._mixed(u) / (6 * h2) + self.k2 * u0 + self._lap(w) / 12).reshape(-1)
        # scheme6: Delta(U + h^2/30 K U) + h^2/6 P(U + h^2/15 K U) + h^4/30 T_x T_y T_z U + K U
        #   + h^2/20 (lap k^2 - k^4) U + h^2/10 sum (k^2)_nu delta_nu (1 + h^2/6 (T_mu + T_rho + K)) U
        v = u + h2 / 30 * w
        y = self._lap(v) / h2 + self._mixed(u + h2 / 15 * w) / (6 * h2)
        y = y + _second(_second(_second(u, 0), 1), 2) / (30 * h2)
        y = y + self.k2 * u0 + h2 / 20 * (self.lap - self.k2 * self.k2) * u0
        for a in range(3):
            o = [b for b in range(3) if b != a]
            n = u.shape[a]
            t = _second(_inner(u, [o[1]]), o[0]) + _second(_inner(u, [o[0]]), o[1])
            t = _inner(u, o) + t / 6 + h2 / 6 * _inner(w, o)
            y = y + h2 / 10 * self.dk[a] * (t.narrow(a, 2, n - 2) - t.narrow(a, 0, n - 2)) / (2 * h)
        return y.reshape(-1)

    def rhs(self, f):
        h2, c = self.h ** 2, f[2:-2, 2:-2, 2:-2]
        if self.order == 2:
            return c.reshape(-1)
        f1 = f[1:-1, 1:-1, 1:-1]
        F = c + self._lap(f1) / 12
        if self.order == 6:
            for a in range(3):
                d4 = _inner(_second(_second(f, a), a), [b for b in range(3) if b != a], 2)
                F = F - d4 / 240
                d1 = (_at(f, _off(a), 2) - _at(f, _off(a, -1), 2)) / (2 * self.h)
                F = F + h2 * h2 / 60 * self.dk[a] * d1
            F = F + self._mixed(f1) / 90 - h2 / 20 * self.k2 * c
        return F.reshape(-1)

    def solve(self, F, tol=1e-13, most=70):
        """Full right-preconditioned GMRES, two Gram-Schmidt passes."""
        beta = torch.linalg.vector_norm(F).item()
        V = torch.empty(most + 1, F.numel(), dtype=C128, device=DEV)
        V[0] = F / beta
        Hm = np.zeros((most + 1, most), complex)
        for j in range(most):
            w = self.matvec(self.precond(V[j]))
            for _ in range(2):
                hj = torch.stack([torch.vdot(V[i], w) for i in range(j + 1)])
                for i in range(j + 1):
                    w.sub_(V[i] * hj[i])
                Hm[:j + 1, j] += hj.cpu().numpy()
            Hm[j + 1, j] = torch.linalg.vector_norm(w).item()
            V[j + 1] = w / Hm[j + 1, j].real
            e = np.zeros(j + 2, complex)
            e[0] = beta
            y = np.linalg.lstsq(Hm[:j + 2, :j + 1], e, rcond=None)[0]
            if np.linalg.norm(e - Hm[:j + 2, :j + 1] @ y) <= tol * beta:
                break
        u = torch.zeros_like(F)
        for i, c in enumerate(y):
            u.add_(V[i] * complex(c))
        return self.precond(u)


def _conv(u, W, b, taps):
    """u (ci, S, S, S) under the weights W (co, ci, taps), zero padding."""
    S = u.shape[-1]
    co, ci = W.shape[:2]
    if taps == 1:
        return (W[:, :, 0] @ u.reshape(ci, -1) + b[:, None]).reshape(co, S, S, S)
    p = torch.nn.functional.pad(u, (1,) * 6)
    out = b[:, None].expand(co, S ** 3)
    for t in range(27):
        dz, dy, dx = t // 9, (t // 3) % 3, t % 3
        out = out + W[:, :, t] @ p[:, dz:dz + S, dy:dy + S, dx:dx + S].reshape(ci, -1)
    return out.reshape(co, S, S, S)


def _network(w, x, S):
    """The encoder-decoder on one sample x (2, S^3), in the precision of its arguments."""
    at, parts = 0, []
    for ci, co, taps, _ in CONVS:
        W = w[at:at + co * ci * taps].reshape(co, ci, taps)
        at += co * ci * taps
        parts.append((W, w[at:at + co], taps))
        at += co
    c = lambda i, u: torch.relu(_conv(u, *parts[i]))  # noqa: E731
    pool = lambda u: torch.nn.functional.avg_pool3d(u[None], 2)[0]  # noqa: E731
    up = lambda u: u.repeat_interleave(2, 1).repeat_interleave(2, 2).repeat_interleave(2, 3)  # noqa: E731
    s1 = c(1, c(0, x.reshape(2, S, S, S)))
    s2 = c(3, c(2, pool(s1)))
    s3 = c(5, c(4, pool(s2)))
    d = c(8, torch.cat([up(c(7, c(6, pool(s3)))), s3]))
    d = c(9, torch.cat([up(d), s2]))
    d = c(10, torch.cat([up(d), s1]))
    return _conv(d, *parts[11]).reshape(2, -1)


def _linear_rows(S, nf):
    """Rows that interpolate the halo grid's values (nf + 4 nodes) at the network's S nodes along one axis."""
    R = np.zeros((S, nf + 4))
    for i in range(S):
        q, r = divmod((i + 1) * (nf + 1), S + 1)
        R[i, q - 1 + 2] += 1 - r / (S + 1)
        R[i, q + 2] += r / (S + 1)
    return torch.from_numpy(R).to(DEV)


def _cubic_rows(nc, nf, gamma):
    """Keys' cubic weights (a = -1/2) of the fine nodes, with ghosts gamma^m of the boundary node."""
    R = np.zeros((nf, nc), complex)
    for o in range(nf):
        q, r = divmod((o + 1) * (nc + 1), nf + 1)
        t = r / (nf + 1)
        w = (-0.5 * t ** 3 + t * t - 0.5 * t, 1.5 * t ** 3 - 2.5 * t * t + 1, -1.5 * t ** 3 + 2 * t * t + 0.5 * t,
             0.5 * t ** 3 - 0.5 * t * t)
        for k in range(4):
            c = q - 2 + k
            m = max(-c, c - nc + 1, 0)
            R[o, min(max(c, 0), nc - 1)] += w[k] * gamma ** m
    return torch.from_numpy(R).to(DEV)


def _apply3(R, u):
    """The 1D matrix R along all three axes."""
    for _ in range(3):
        u = torch.tensordot(u, R, dims=([0], [1]))
    return u


def exact(case, seed):
    kind = case["kind"]
    if kind in ("solve", "medium"):
        n3, h, k2, f = _problem(case, seed)
        E = _Exact(k2, n3, h, case["order"], case["k0"])
        return E.solve(E.rhs(f))
    if kind == "direct":
        n3 = (case["nz"], case["ny"], case["nx"])
        h = 1.0 / max(n3)
        E = _Exact(_medium("constant", n3, h, case["k0"], seed), n3, h, 2, case["k0"])
        return E.precond(_wavy(n3, case["k0"] * h, seed))
    if kind == "operator":
        n3 = (case["nz"], case["ny"], case["nx"])
        h = 1.0 / (max(n3) + 1)
        k2 = _medium("inclusions", n3, h, case["k0"], seed)
        E = _Exact(k2, n3, h, case["order"], case["k0"])
        return {"F": E.rhs(_wave(k2, case["k0"], n3, h, _dirs(1, seed)[0])),
                "y": E.matvec(_wavy(n3, case["k0"] * h, seed))}
    if kind == "waves":
        n3, h = (case["n"],) * 3, 1.0 / (case["n"] + 1)
        k2 = _medium("inclusions", n3, h, case["k0"], seed)
        E = _Exact(k2, n3, h, 6, case["k0"])
        return [E.solve(E.rhs(_wave(k2, case["k0"], n3, h, d))) for d in _dirs(case["count"], seed)]
    if kind == "uneven":
        out = []
        for p, (n, k0) in enumerate(_uneven(case, seed)):
            n3, h = (n, n, n), 1.0 / (n + 1)
            E = _Exact(_medium("inclusions", n3, h, k0, (seed, p)), n3, h, 6, k0)
            out.append(E.solve(E.rhs(_gauss(n3, h, (seed, p)))))
        return out
    S = case["size"]
    w = _weights(seed).double().to(DEV)
    if kind == "infer":
        k2, f = _infer_data(case, seed)
        R = _linear_rows(S, case["nf"])
        x = torch.stack([(_apply3(R, k2) / NET_K0 ** 2 - 1).reshape(-1), _apply3(R, f.real.contiguous()).reshape(-1)])
        y = _network(w, x, S)
        C = _cubic_rows(S, case["nf"], _gamma(NET_K0, 1.0 / (S + 1)))
        return {"y": y[None], "x0": _apply3(C, torch.complex(y[0], y[1]).reshape(S, S, S)).reshape(-1)}
    w.requires_grad_(True)
    x, t = _train_data(case, seed)
    N, loss = t.numel(), 0.0
    for b in range(case["batch"]):       # one sample at a time: the 64-bit activations of one are a few GB
        l = ((_network(w, x[b].double(), S) - t[b].double()) ** 2).sum() / N
        l.backward()
        loss += l.item()
    return {"loss": loss, "grads": w.grad.clone()}
