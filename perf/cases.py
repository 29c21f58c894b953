"""What a user of this framework has it do, as cases that can be timed and checked.

A case is a dict of plain values.  `prepare` builds what a simulation program
holds before it steps (a context with its opacity and inflow, an initial state
on the GPU), `run` takes one pass through the public entry points (set the
state, advance it, read it back), `work` states the bytes and operations the
pass cannot do without, and `exact` gives what `run` returns in plain 64-bit
torch.  States are smooth heated fronts running into cold material -- the shape
every workload of this framework develops from its hot inflow edge -- with the
front's place and width, its anisotropy and the opacity seeded.
"""
import ctypes
import math

import numpy as np
import torch

from paper_1811_05579_amd import Grte, Grte2D, GrteBatch, GrteDiff, Mlp, load, step_group

DEV = "cuda"
F64 = torch.float64
GROUP_EPS = (1.0, 1e-2, 1e-4)          # the three scaling regimes run side by side
PARAMS, HIDDEN, FEATURES = 4609, 64, 5  # the learned guess network 5-64-64-1
BATCH_NV = (8, 16, 32, 64)


def listed():
    return [
        # the smallest simulation: a thin slab at a low quadrature order, where launches and latency count
        dict(name="slab-100x16", kind="slab", nx=100, nv=16, law=0, eps=1e-2, fp32=False, steps=20),
        # an ordinary single slab, odd size, temperature-dependent opacity, intensities stored in binary32
        dict(name="slab-1543x32-f32", kind="slab", nx=1543, nv=32, law=3, eps=1e-3, fp32=True, steps=10),
        # the largest slab: transport, intermediate and diffusive runs advanced together by one grouped launch
        dict(name="group-3x4096x64", kind="group", nx=4096, nv=64, steps=10),
        # the implicit reference solver a user checks a run against (iterated nonlinear opacity)
        dict(name="reference-512x32", kind="reference", nx=512, nv=32, eps=0.5),
        # a small parameter study: a few uneven slabs as one ensemble, stepped through the captured graph
        dict(name="batch-24", kind="batch", slabs=24, fp32=False, steps=10),
        # the throughput workload: thousands of uneven slabs, binary32 intensities
        dict(name="batch-4096-f32", kind="batch", slabs=4096, fp32=True, steps=4),
        # a small ragged rectangle, temperature-dependent opacity: a 2-D set-up being tried out
        dict(name="plane-47x33x8", kind="plane", nx=47, ny=33, nv=8, law=3, eps=1e-2, hi=3.0, fp32=False, steps=3),
        # two materials of very different opacity in the diffusive regime, many directions
        dict(name="plane-512x512x64", kind="plane", nx=512, ny=512, nv=64, law=0, eps=1e-4, hi=1000.0, fp32=False,
             steps=3),
        # the largest rectangle, binary32 intensities
        dict(name="plane-1024x1024x32-f32", kind="plane", nx=1024, ny=1024, nv=32, law=0, eps=1e-3, hi=100.0,
             fp32=True, steps=2),
        # fitting the learned guess to logged steps (forward, backward, Adam)
        dict(name="guess-train-4096", kind="train", rows=20000, batch=4096, steps=20),
        # evaluating it for every cell of a large rectangle
        dict(name="guess-predict-1m", kind="predict", rows=1 << 20),
        # the diffusion-limit scheme that thick runs are compared with
        dict(name="diffusion-1000", kind="diffusion", nx=1000, law=3, scheme=0, steps=50),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["slab", "slab", "group", "reference", "batch", "batch", "plane", "plane", "train", "predict",
                       "diffusion"])
    if kind == "slab":
        return dict(kind=kind, nx=_log_int(rng, 20, 4096), nv=rng.choice([4, 8, 14, 16, 32, 50, 64]),
                    law=rng.choice([0, 3]), eps=10 ** rng.uniform(-4, 0), fp32=rng.random() < 0.4,
                    steps=rng.randint(4, 20))
    if kind == "group":
        return dict(kind=kind, nx=_log_int(rng, 200, 4096), nv=rng.choice([16, 32, 64]), steps=rng.randint(4, 10))
    if kind == "reference":
        return dict(kind=kind, nx=_log_int(rng, 60, 1000), nv=rng.choice([8, 16, 32]), eps=10 ** rng.uniform(-1, 0))
    if kind == "batch":
        return dict(kind=kind, slabs=_log_int(rng, 8, 4000), fp32=rng.random() < 0.5, steps=rng.randint(2, 4))
    if kind == "plane":
        nv = rng.choice([8, 16, 32, 64])
        side = _log_int(rng, 24, 700 if nv <= 32 else 500)
        return dict(kind=kind, nx=side, ny=max(8, int(side * rng.uniform(0.6, 1.0))), nv=nv, law=rng.choice([0, 0, 3]),
                    eps=10 ** rng.uniform(-3.5, -1), hi=10 ** rng.uniform(0, 2.5), fp32=rng.random() < 0.5,
                    steps=rng.randint(1, 2))
    if kind == "train":
        return dict(kind=kind, rows=_log_int(rng, 3000, 100000), batch=_log_int(rng, 256, 8192),
                    steps=rng.randint(5, 20))
    if kind == "predict":
        return dict(kind=kind, rows=_log_int(rng, 500, 1 << 20))
    return dict(kind=kind, nx=_log_int(rng, 50, 4096), law=rng.choice([0, 3]), scheme=rng.choice([0, 1]),
                steps=rng.randint(10, 50))


# ---------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------
def _rng(seed):
    return np.random.default_rng(181105579 + seed)


def _gauss(nv):
    x, w = np.polynomial.legendre.leggauss(nv)
    return np.ascontiguousarray(x[x > 0]), np.ascontiguousarray(w[x > 0])


def _up(x):
    return torch.as_tensor(np.ascontiguousarray(x), dtype=F64, device=DEV)


def _front(x, place, width, cold=1e-2):
    return cold + 0.5 * (1.0 - cold) * (1.0 - torch.tanh((x - place) / width))


def _slab_inputs(nx, nv, law, eps, rng):
    """One slab: (mu, omega, sigma0, bL, bR) on the host, (E, O, T) on the GPU; a = c = Cv = L = 1."""
    mu, om = _gauss(nv)
    P = mu.size
    sigma0 = rng.uniform(0.5, 2.0, nx)
    bL, bR = rng.uniform(0.9, 1.1, P), np.zeros(P)
    place, width, amp = rng.uniform(0.2, 0.5), rng.uniform(0.03, 0.1), rng.uniform(0.02, 0.1)
    x = (torch.arange(nx, dtype=F64, device=DEV) + 0.5) / nx
    m = _up(mu)
    T = _front(x, place, width)
    E = (T ** 4)[:, None] * (1.0 + amp * min(1.0, eps) * (1.5 * m ** 2 - 0.5) * torch.sin(7.0 * x + amp)[:, None])
    K = 0.5 * (T[1:] ** law + T[:-1] ** law)
    O = torch.zeros(nx + 1, P, dtype=F64, device=DEV)
    # the diffusive flux, bounded where the slab is thin
    O[1:-1] = -(K / (10.0 * eps * eps * K + 1.0))[:, None] * m * (E[1:] - E[:-1]) * nx
    O[0], O[-1] = O[1], O[-2]
    return mu, om, sigma0, bL, bR, E.contiguous(), O, T


class _Member:
    """One slab of an ensemble, as GrteBatch takes it."""

    L = a = c = Cv = 1.0
    m = 3


def _members(slabs, fp32):
    """The ensemble's slabs: sizes, orders, eps and opacity are the study's own, not the seed's.  Binary32
    ensembles reach an order further into the diffusive regime, where O carries few digits either way."""
    rng = np.random.default_rng(4096 + slabs)
    nx, nv = rng.integers(64, 2049, slabs), rng.choice(BATCH_NV, slabs)
    eps, sig = 10.0 ** rng.uniform(-5 if fp32 else -4, 0, slabs), 10.0 ** rng.uniform(-1, 2, slabs)
    grids = {int(n): _gauss(int(n)) for n in BATCH_NV}
    out = []
    for i in range(slabs):
        w = _Member()
        w.N, (w.mu, w.omega), w.eps, w.sig = int(nx[i]), grids[int(nv[i])], float(eps[i]), float(sig[i])
        w.P, w.dt = w.mu.size, 0.5 / w.N
        out.append(w)
    return out


def _batch_inputs(members, rng):
    """Packed (sigma0, bL, bR) on the host and (E, O, T) on the GPU, formed for all slabs at once."""
    n = len(members)
    N, P = np.array([w.N for w in members]), np.array([w.P for w in members])
    par = [_up(v) for v in (rng.uniform(0.2, 0.5, n), rng.uniform(0.03, 0.1, n), rng.uniform(0.02, 0.1, n),
                            [w.eps for w in members], [w.sig for w in members])]
    Nd, Pd = torch.as_tensor(N, device=DEV), torch.as_tensor(P, device=DEV)
    mus = _up(np.concatenate([w.mu for w in members]))
    off = torch.cumsum(Pd, 0) - Pd

    def owner(sizes):
        who = torch.repeat_interleave(torch.arange(n, device=DEV), sizes)
        return who, torch.arange(int(sizes.sum()), device=DEV) - (torch.cumsum(sizes, 0) - sizes)[who]

    def temp(who, x):
        return _front(x, par[0][who], par[1][who])

    def even(who, x, m):                   # E at position x of slab `who` for ordinate m
        amp = par[2][who]
        return temp(who, x) ** 4 * (1.0 + amp * torch.clamp(par[3][who], max=1.0) * (1.5 * m * m - 0.5)
                                    * torch.sin(7.0 * x + amp))

    who, j = owner(Nd)
    T = temp(who, (j + 0.5) / Nd[who])
    who, k = owner(Nd * Pd)
    m = mus[off[who] + k % Pd[who]]
    E = even(who, (k // Pd[who] + 0.5) / Nd[who], m)
    del who, k, m
    who, k = owner((Nd + 1) * Pd)
    m = mus[off[who] + k % Pd[who]]
    h = 1.0 / Nd[who]
    x = (k // Pd[who]) * h
    K = temp(who, x) ** 3
    O = -K / (10.0 * par[3][who] ** 2 * K + par[4][who]) * m * (even(who, x + 0.5 * h, m) - even(who, x - 0.5 * h, m)) / h
    sigma0 = np.repeat([w.sig for w in members], N)
    bL = rng.uniform(0.9, 1.1, int(P.sum()))
    return sigma0, bL, np.zeros_like(bL), E, O, T


def _circle(nv):
    th = 2.0 * np.pi * (np.arange(nv // 2) + 0.5) / nv
    return np.cos(th), np.sin(th), np.full(nv // 2, 2.0 / nv)


def _plane_inputs(case, rng):
    """One rectangle [0, 1]^2: (mu, eta, omega, b) on the host, (sigma0, E, Ox, Oy, T) on the GPU.  The
    opacity is 1 or `hi` on the cells nearest to 64 seeded sites."""
    nx, ny, eps, law = case["nx"], case["ny"], case["eps"], case["law"]
    mu, eta, om = _circle(case["nv"])
    P = mu.size
    b = np.zeros((4, P))
    b[0] = rng.uniform(0.9, 1.1, P)
    sites, kind = _up(rng.uniform(0, 1, (64, 2))), rng.random(64) < 0.5
    value = _up(np.where(kind, 1.0, case["hi"]))
    place, width, amp, phase = rng.uniform(0.1, 0.25), rng.uniform(0.03, 0.06), rng.uniform(0.02, 0.1), rng.uniform(0, 6)
    x = ((torch.arange(nx, dtype=F64, device=DEV) + 0.5) / nx)[None, :]
    y = ((torch.arange(ny, dtype=F64, device=DEV) + 0.5) / ny)[:, None]
    best, sigma = torch.full((ny, nx), 1e9, dtype=F64, device=DEV), torch.ones(ny, nx, dtype=F64, device=DEV)
    for k in range(64):
        d2 = (x - sites[k, 0]) ** 2 + (y - sites[k, 1]) ** 2
        near = d2 < best
        best, sigma = torch.where(near, d2, best), torch.where(near, value[k], sigma)
    T = _front(x, place + 0.04 * torch.sin(4.0 * y + phase), width)
    m, e = _up(mu), _up(eta)
    E = (T ** 4)[..., None] * (1.0 + amp * min(1.0, eps) * m * m * torch.cos(5.0 * x + 3.0 * y)[..., None])
    K = T ** law
    D = (K / (10.0 * eps * eps * K + sigma))[..., None]
    gx, gy = torch.zeros_like(E), torch.zeros_like(E)
    gx[:, 1:-1] = (E[:, 2:] - E[:, :-2]) * (0.5 * nx)
    gy[1:-1] = (E[2:] - E[:-2]) * (0.5 * ny)
    F = -D * (m * gx + e * gy)
    Ox, Oy = torch.zeros(ny, nx + 1, P, dtype=F64, device=DEV), torch.zeros(ny + 1, nx, P, dtype=F64, device=DEV)
    Ox[:, 1:-1] = 0.5 * (F[:, 1:] + F[:, :-1])
    Oy[1:-1] = 0.5 * (F[1:] + F[:-1])
    return mu, eta, om, b, sigma.contiguous(), E.contiguous(), Ox, Oy, T.contiguous()


def _theta(rng):
    parts = [rng.uniform(-1, 1, HIDDEN * FEATURES) / math.sqrt(FEATURES), rng.uniform(-0.1, 0.1, HIDDEN),
             rng.uniform(-1, 1, HIDDEN * HIDDEN) / 8.0, rng.uniform(-0.1, 0.1, HIDDEN), rng.uniform(-1, 1, HIDDEN) / 8.0,
             rng.uniform(-0.1, 0.1, 1)]
    return np.concatenate(parts).astype(np.float32)


def _rows(n, rng):
    """Training rows as logged steps give them: log10 of rho*, T, sigma, eps and dt, and log(T_new / T)."""
    lt = rng.uniform(-2, 0, n)
    rho, sig = 4 * lt + rng.normal(0, 0.3, n), rng.uniform(-0.3, 6.0, n)
    f = np.stack([rho, lt, sig, rng.uniform(-4, 0, n), rng.uniform(-4, -2, n)], 1)
    target = 0.05 * (rho - 4 * lt) + 0.02 * np.sin(sig) + 0.002 * rng.normal(size=n)
    return np.concatenate([f, target[:, None]], 1).astype(np.float32)


def _norm(rows):
    r = rows.astype(np.float64)
    mean, sd = r.mean(0), r.std(0)
    return np.concatenate([mean[:5], sd[:5], mean[5:], sd[5:]]).astype(np.float32)


def _diffusion_inputs(case, rng):
    x = (np.arange(case["nx"]) + 0.5) / case["nx"]
    T = 0.1 + 0.45 * (1.0 - np.tanh((x - rng.uniform(0.3, 0.6)) / rng.uniform(0.05, 0.15)))
    return rng.uniform(0.5, 2.0, case["nx"]), T


# ---------------------------------------------------------------------------
# passes
# ---------------------------------------------------------------------------
def prepare(case, seed):
    rng, kind = _rng(seed), case["kind"]
    if kind in ("slab", "group", "reference"):
        law, eps = case.get("law", 3), case.get("eps", 1e-2)
        s = dict(kind=kind, dt=0.5 / case["nx"], eps=eps, steps=case.get("steps", 1), fp32=case.get("fp32", False),
                 ctx=[], state=[], out=[])
        for e in GROUP_EPS if kind == "group" else (eps,):
            mu, om, sigma0, bL, bR, E, O, T = _slab_inputs(case["nx"], case["nv"], law, e, rng)
            g = Grte(case["nx"], mu, om, opacity_law=law)
            g.set_opacity(sigma0)
            g.set_inflow(bL, bR)
            if case.get("fp32"):
                g.set_storage(True)
            s["ctx"].append(g)
            s["state"].append((E, O, T))
            s["out"].append(tuple(torch.empty_like(v) for v in (E, O, T)))
        return s
    if kind == "batch":
        members = _members(case["slabs"], case["fp32"])
        sigma0, bL, bR, E, O, T = _batch_inputs(members, rng)
        g = GrteBatch(members)
        g.set_opacity(sigma0)
        g.set_inflow(bL, bR)
        g.set_storage(case["fp32"])
        g.use_graph(True)
        return dict(kind=kind, steps=case["steps"], fp32=case["fp32"], ctx=g, state=(E, O, T),
                    out=tuple(torch.empty_like(v) for v in (E, O, T)))
    if kind == "plane":
        mu, eta, om, b, sigma0, E, Ox, Oy, T = _plane_inputs(case, rng)
        g = Grte2D(case["nx"], case["ny"], mu, eta, om, opacity_law=case["law"])
        g.set_opacity(sigma0)
        g.set_inflow(b)
        if case["fp32"]:
            g.set_storage(True)
        state = (E, Ox, Oy, T)
        return dict(kind=kind, steps=case["steps"], dt=0.5 / max(case["nx"], case["ny"]), eps=case["eps"],
                    fp32=case["fp32"], ctx=g, state=state, out=tuple(torch.empty_like(v) for v in state))
    if kind in ("train", "predict"):
        rows, theta = _rows(case["rows"], rng), _theta(rng)
        m = Mlp()
        m.set_params(theta)
        m.set_norm(_norm(rows))
        return dict(kind=kind, ctx=m, theta=theta, rows=torch.from_numpy(rows).to(DEV), batch=case.get("batch"),
                    steps=case.get("steps"))
    sigma0, T = _diffusion_inputs(case, rng)
    g = GrteDiff(case["nx"], opacity_law=case["law"])
    g.set_opacity(sigma0)
    return dict(kind=kind, ctx=g, T=_up(T), dt=2e-4, scheme=case["scheme"], steps=case["steps"])


def _kept(out, fp32):
    """The outputs as a program keeps them: intensities stored in binary32 hold no more than that."""
    return tuple(v.float() for v in out[:-1]) + out[-1:] if fp32 else out


def _read_on_device(call, ctx, out):
    """State readout into device memory, through the C entry point (the classes of the binding copy to the host)."""
    status = call(ctx._h, *[ctypes.c_void_p(v.data_ptr()) for v in out], 1)
    if status != 0:
        raise RuntimeError("state readout: status %d" % status)


def run(s):
    kind, g = s["kind"], s["ctx"]
    if kind in ("slab", "group", "reference"):
        for c, state in zip(g, s["state"]):
            c.set_state(*state)
        if kind == "reference":
            g[0].reference_step(s["dt"], s["eps"])
        elif kind == "group":
            for _ in range(s["steps"]):
                step_group(g, [s["dt"]] * len(g), GROUP_EPS)
        else:
            for _ in range(s["steps"]):
                g[0].step(s["dt"], s["eps"])
        for c, out in zip(g, s["out"]):
            c.get_state(out)
        return [_kept(out, s["fp32"]) for out in s["out"]]
    if kind == "batch":
        g.set_state(*s["state"])
        for _ in range(s["steps"]):
            g.step()
        _read_on_device(load().grte_batch_get_state, g, s["out"])
        return _kept(s["out"], s["fp32"])
    if kind == "plane":
        g.set_state(*s["state"])
        for _ in range(s["steps"]):
            g.step(s["dt"], s["eps"])
        _read_on_device(load().grte2d_get_state, g, s["out"])
        return _kept(s["out"], s["fp32"])
    if kind == "train":
        g.set_params(s["theta"])
        loss = g.train(s["rows"], s["steps"], batch=s["batch"])
        return loss, g.get_params()[0]
    if kind == "predict":
        return g.predict(s["rows"])
    g.set_state(s["T"])
    for _ in range(s["steps"]):
        g.step(s["dt"], scheme=s["scheme"])
    return g.get_state()


def work(case):
    """Per step: the stored state read once and written once; about 40 operations per cell and pair for the two
    linear solves of a step done by elimination."""
    kind, n = case["kind"], case.get("steps", 1)
    wide = 4 if case.get("fp32") else 8
    if kind in ("slab", "group", "reference"):
        N, P, k = case["nx"], case["nv"] // 2, len(GROUP_EPS) if kind == "group" else 1
        return dict(bytes=n * k * 2 * (wide * (2 * N + 1) * P + 8 * N), flops=n * k * 40 * N * P)
    if kind == "batch":
        cells = sum(w.N for w in _members(case["slabs"], case["fp32"]))
        pairs = sum(w.N * w.P for w in _members(case["slabs"], case["fp32"]))
        return dict(bytes=n * 2 * (wide * 2 * pairs + 8 * cells), flops=n * 40 * pairs)
    if kind == "plane":
        N, P = case["nx"] * case["ny"], case["nv"] // 2
        return dict(bytes=n * 2 * (wide * 3 * N * P + 8 * N), flops=n * 80 * N * P)
    if kind == "train":
        used = case["steps"] * min(case["batch"], case["rows"])
        return dict(bytes=24 * used + 16 * PARAMS * case["steps"], flops=6 * PARAMS * used)
    if kind == "predict":
        return dict(bytes=28 * case["rows"], flops=2 * PARAMS * case["rows"])
    return dict(bytes=n * 16 * case["nx"], flops=n * 60 * case["nx"])


# ---------------------------------------------------------------------------
# the same results in plain 64-bit torch
# ---------------------------------------------------------------------------
def _tri(a, b, c, d):
    """Tridiagonal systems along the last axis by parallel cyclic reduction (a: sub-, c: super-diagonal)."""
    def left(v, k, fill):
        return torch.cat([torch.full_like(v[..., :k], fill), v[..., :-k]], -1)

    def right(v, k, fill):
        return torch.cat([v[..., k:], torch.full_like(v[..., :k], fill)], -1)

    a, b, c, d = torch.broadcast_tensors(a, b, c, d)
    k, n = 1, b.shape[-1]
    while k < n:
        p, q = -a / left(b, k, 1.0), -c / right(b, k, 1.0)
        a, b, c, d = (p * left(a, k, 0.0), b + p * left(c, k, 0.0) + q * right(a, k, 0.0), q * right(c, k, 0.0),
                      d + p * left(d, k, 0.0) + q * right(d, k, 0.0))
        k *= 2
    return d / b


def _root(q4, lin, rhs, T):
    """The root of q4 T^4 + lin (T - T_n) = rhs by Newton from above it (convex, increasing)."""
    C = rhs + lin * T
    top = torch.minimum(C.clamp(min=0) / lin, (C.clamp(min=0) / q4.clamp(min=1e-300)) ** 0.25)
    x = torch.maximum(top, 1e-30 * torch.ones_like(top))
    for _ in range(60):
        x = x - (q4 * x ** 4 + lin * x - C) / (4 * q4 * x ** 3 + lin)
    return x


class _Slab:
    """The 1-D step on (pair, cell) arrays; a = c = Cv = L = 1."""

    def __init__(self, mu, om, sigma0, bL, bR, law, dt, eps):
        self.mu, self.om, self.bL, self.bR = (_up(v)[:, None] for v in (mu, om, bL, bR))
        self.s, self.law, self.dt, self.eps = _up(sigma0), law, dt, eps
        self.N = self.s.numel()
        sl, sr = self.s[:-1], self.s[1:]
        self.sn = 2 * sl * sr / (sl + sr)

    def operator(self, K):
        N, e2, dt = self.N, self.eps ** 2, self.dt
        Kn = 0.5 * (K[1:] + K[:-1])
        den = Kn * e2 + self.sn * dt
        aw, bc = Kn * e2 / den, Kn * dt * N / den
        h = K * e2 * dt * N
        up, lo = torch.zeros_like(K), torch.zeros_like(K)
        up[:-1], lo[1:] = h[:-1] * bc, h[1:] * bc
        up[0] *= 2
        lo[-1] *= 2
        bd = torch.zeros_like(K)
        bd[0], bd[-1] = 2 * h[0] / self.eps, 2 * h[-1] / self.eps
        return aw, bc, h, lo, up, bd

    def nodes(self, E, On, aw, bc):
        inner = aw * On[:, 1:-1] - bc * self.mu * (E[:, 1:] - E[:, :-1])
        k = 2 / self.eps
        return torch.cat([k * (self.bL - E[:, :1]) - inner[:, :1], inner,
                          k * (E[:, -1:] - self.bR) - inner[:, -1:]], 1)

    def rhs(self, En, On, K, aw, h, src):
        f = torch.zeros(On.shape, dtype=F64, device=DEV)
        f[:, 1:-1] = aw * On[:, 1:-1]
        d = f[:, 1:] - f[:, :-1]
        d[:, 0] *= 2
        d[:, -1] *= 2
        r = K * self.eps ** 2 * En + src - h * self.mu * d
        k = 2 * h / self.eps
        r[:, :1] += k[0] * self.mu * self.bL
        r[:, -1:] += k[-1] * self.mu * self.bR
        return r

    def solve(self, lam, op, m1, m2, d):
        lo, up, bd = op[3], op[4], op[5]
        return _tri(-m2 * lo, lam + m2 * (lo + up) + m1 * bd, -m2 * up, d)

    def predict(self, En, On, Tn, K):
        """E*, O*, rho* and beta of the prediction with K given per cell."""
        dt, e2, mu, om = self.dt, self.eps ** 2, self.mu, self.om
        beta = 4 * self.s * dt * (Tn ** 3 if self.law == 0 else 1.0) / e2
        op = self.operator(K)
        aw, bc, h = op[:3]
        lam = K * e2 + self.s * dt
        low = K * e2 + self.s * dt / (1 + beta)
        r = self.rhs(En, On, K, aw, h, self.s * dt * Tn ** 4 / (1 + beta))
        lo, up, bd = op[3:]
        W, M1, M2 = om.sum(), (om * mu).sum(), (om * mu * mu).sum()
        rho = (om * En).sum(0)

        def apart(rho):                      # E_p - rho, from the residual of the isotropic state
            d = torch.zeros(self.N + 1, dtype=F64, device=DEV)
            d[1:-1] = rho[1:] - rho[:-1]
            L = lo * d[:-1] - up * d[1:]
            return self.solve(lam, op, mu, mu * mu, r - low * rho - mu * mu * L - mu * bd * rho)

        for _ in range(200):
            res = (om * apart(rho)).sum(0) - (1 - W) * rho
            z = res + self.solve(low, op, M1, M2, (lam - low) * res)
            rho = rho + z
            if float(z.abs().max()) <= 1e-15 * float(rho.abs().max()):
                break
        E = rho + apart(rho)
        return E, self.nodes(E, On, aw, bc), (om * E).sum(0), beta

    def step(self, En, On, Tn):
        dt, e2, s = self.dt, self.eps ** 2, self.s
        Es, Os, rs, beta = self.predict(En, On, Tn, Tn ** self.law)
        D = (self.om * self.mu * (Os[:, 1:] - Os[:, :-1])).sum(0) * self.N
        us = (Tn ** 4 + beta * rs) / (1 + beta)
        Ks = us.clamp(min=0) ** 0.75 if self.law == 3 else torch.ones_like(us)
        T = _root(s * dt, e2 * Ks + s * dt, s * dt * ((self.om * En).sum(0) - dt * D), Tn)
        K = T ** self.law
        op = self.operator(K)
        E = self.solve(K * e2 + s * dt, op, self.mu, self.mu ** 2, self.rhs(En, On, K, op[0], op[2], s * dt * T ** 4))
        return E, self.nodes(E, On, op[0], op[1]), T

    def reference(self, En, On, Tn):
        T = Tn
        for _ in range(500):
            Es, Os, rs, beta = self.predict(En, On, Tn, T ** self.law)
            last, T = T, ((Tn ** 4 + beta * rs) / (1 + beta)).clamp(min=0) ** 0.25
            if float((T - last).abs().max()) <= 1e-14 * float(T.max()):
                break
        return Es, Os, T


def _slab_exact(data, law, dt, eps, steps, reference=False):
    mu, om, sigma0, bL, bR, E, O, T = data
    S, E, O = _Slab(mu, om, sigma0, bL, bR, law, dt, eps), E.T.contiguous(), O.T.contiguous()
    for _ in range(steps):
        E, O, T = S.reference(E, O, T) if reference else S.step(E, O, T)
    return E.T.contiguous(), O.T.contiguous(), T


class _Plane:
    """The 2-D step with dense matrices per pair (small rectangles); a = c = Cv = 1 on [0, 1]^2."""

    def __init__(self, case, mu, eta, om, b, sigma0):
        self.nx, self.ny, self.law, self.eps = case["nx"], case["ny"], case["law"], case["eps"]
        self.dt = 0.5 / max(self.nx, self.ny)
        self.mu, self.eta, self.om = (_up(v) for v in (mu, eta, om))
        self.P, self.N = mu.size, self.nx * self.ny
        self.b, self.s = _up(b), sigma0
        eye = torch.eye(self.N, dtype=F64, device=DEV).reshape(self.ny, self.nx, self.N)
        (self.gxx, self.gxy), (self.gyx, self.gyy) = self.gradients(eye)

    def gradients(self, X):
        """(d_x, d_y) of X (ny, nx, ...) at the interior x-faces and y-faces."""
        def along(v, n, dim):
            v = v.movedim(dim, 0)
            d = torch.empty_like(v)
            d[1:-1] = (v[2:] - v[:-2]) * (0.5 * n)
            d[0], d[-1] = (v[1] - v[0]) * n, (v[-1] - v[-2]) * n
            return d.movedim(0, dim)

        cx, cy = along(X, self.nx, 1), along(X, self.ny, 0)
        x = (X[:, 1:] - X[:, :-1]) * self.nx, 0.5 * (cy[:, 1:] + cy[:, :-1])
        y = 0.5 * (cx[1:] + cx[:-1]), (X[1:] - X[:-1]) * self.ny
        return x, y

    def faces(self, K):
        def harm(p, q):
            return 2 * p * q / (p + q)

        e2, dt, s = self.eps ** 2, self.dt, self.s
        out = []
        for Kf, sf in ((0.5 * (K[:, 1:] + K[:, :-1]), harm(s[:, 1:], s[:, :-1])),
                       (0.5 * (K[1:] + K[:-1]), harm(s[1:], s[:-1]))):
            den = Kf * e2 + sf * dt
            out.append((Kf * e2 / den, Kf * dt / den))
        return out

    def fluxes(self, p, X, inner_x, inner_y, inflow):
        """All faces' O of pair p from the interior ones and the inflow relations for cell values X."""
        sx, sy = math.copysign(1.0, float(self.mu[p])), math.copysign(1.0, float(self.eta[p]))
        k, b = 2 / self.eps, self.b[:, p] * inflow
        l = sx * k * (b[0] - X[:, :1]) - inner_x[:, :1]
        r = -sx * k * (b[1] - X[:, -1:]) - inner_x[:, -1:]
        lo = sy * k * (b[2] - X[:1]) - inner_y[:1]
        hi = -sy * k * (b[3] - X[-1:]) - inner_y[-1:]
        return torch.cat([l, inner_x, r], 1), torch.cat([lo, inner_y, hi], 0)

    def divergence(self, p, Fx, Fy):
        return self.mu[p] * (Fx[:, 1:] - Fx[:, :-1]) * self.nx + self.eta[p] * (Fy[1:] - Fy[:-1]) * self.ny

    def system(self, K, lam, En, Oxn, Oyn, src):
        """Inverses of the per-pair matrices and the right-hand sides (pair, cell)."""
        (ax, gx), (ay, gy) = self.faces(K)
        e2 = self.eps ** 2
        k = K * e2 * self.dt
        eye = torch.eye(self.N, dtype=F64, device=DEV).reshape(self.ny, self.nx, self.N)
        inv, rhs = [], []
        zero = torch.zeros(self.ny, self.nx, dtype=F64, device=DEV)
        for p in range(self.P):
            m, e = self.mu[p], self.eta[p]
            Fx = -gx[..., None] * (m * self.gxx + e * self.gxy)
            Fy = -gy[..., None] * (m * self.gyx + e * self.gyy)
            A = k[..., None] * self.divergence(p, *self.fluxes(p, eye, Fx, Fy, 0.0))
            A = A.reshape(self.N, self.N) + torch.diag(lam.reshape(-1))
            inv.append(torch.linalg.inv(A))
            known = self.divergence(p, *self.fluxes(p, zero, ax * Oxn[:, 1:-1, p], ay * Oyn[1:-1, :, p], 1.0))
            rhs.append((K * e2 * En[..., p] + src - k * known).reshape(-1))
        return inv, rhs, (ax, gx, ay, gy)

    def all_fluxes(self, E, Oxn, Oyn, face):
        ax, gx, ay, gy = face
        (xx, xy), (yx, yy) = self.gradients(E)
        Ox, Oy = torch.empty_like(Oxn), torch.empty_like(Oyn)
        for p in range(self.P):
            m, e = self.mu[p], self.eta[p]
            ix = ax * Oxn[:, 1:-1, p] - gx * (m * xx[..., p] + e * xy[..., p])
            iy = ay * Oyn[1:-1, :, p] - gy * (m * yx[..., p] + e * yy[..., p])
            Ox[..., p], Oy[..., p] = self.fluxes(p, E[..., p], ix, iy, 1.0)
        return Ox, Oy

    def cells(self, v):
        return torch.stack(v, -1).reshape(self.ny, self.nx, self.P)

    def step(self, En, Oxn, Oyn, Tn):
        dt, e2, s = self.dt, self.eps ** 2, self.s
        beta = 4 * s * dt * (Tn ** 3 if self.law == 0 else 1.0) / e2
        K = Tn ** self.law
        lam, G = K * e2 + s * dt, (s * dt * beta / (1 + beta)).reshape(-1)
        inv, rhs, face = self.system(K, lam, En, Oxn, Oyn, s * dt * Tn ** 4 / (1 + beta))
        S = torch.eye(self.N, dtype=F64, device=DEV) - sum(w * A for w, A in zip(self.om, inv)) * G
        rho = torch.linalg.solve(S, sum(w * (A @ r) for w, A, r in zip(self.om, inv, rhs)))
        Es = self.cells([A @ (r + G * rho) for A, r in zip(inv, rhs)])
        del inv, S
        Fx, Fy = self.all_fluxes(Es, Oxn, Oyn, face)
        D = sum(self.om[p] * self.divergence(p, Fx[..., p], Fy[..., p]) for p in range(self.P))
        us = (Tn ** 4 + beta * (Es @ self.om)) / (1 + beta)
        Ks = us.clamp(min=0) ** 0.75 if self.law == 3 else torch.ones_like(us)
        T = _root(s * dt, e2 * Ks + s * dt, s * dt * (En @ self.om - dt * D), Tn)
        K = T ** self.law
        inv, rhs, face = self.system(K, K * e2 + s * dt, En, Oxn, Oyn, s * dt * T ** 4)
        E = self.cells([A @ r for A, r in zip(inv, rhs)])
        return (E, *self.all_fluxes(E, Oxn, Oyn, face), T)


def _bf16(theta):
    return torch.as_tensor(theta).to(torch.bfloat16).to(F64).to(DEV)


def _split(th):
    return (th[:320].reshape(HIDDEN, FEATURES), th[320:384], th[384:4480].reshape(HIDDEN, HIDDEN), th[4480:4544],
            th[4544:4608], th[4608])


def _net(th, x):
    W1, b1, W2, b2, W3, b3 = _split(th)
    gelu = torch.nn.functional.gelu
    return gelu(gelu(x @ W1.T + b1) @ W2.T + b2) @ W3 + b3


def _train_exact(theta, rows, norm, batch, steps, lr=1e-3):
    th, data, nm = _up(theta), _up(rows), _up(norm)
    x, y = (data[:, :5] - nm[:5]) / nm[5:10], (data[:, 5] - nm[10]) / nm[11]
    n = len(rows)
    B = min(batch, n)
    m, v, loss = torch.zeros_like(th), torch.zeros_like(th), []
    for k in range(steps):
        at = (k * B + torch.arange(B, device=DEV)) % n
        q = th.clone().requires_grad_(True)
        L = ((_net(q, x[at]) - y[at]) ** 2).mean()
        L.backward()
        loss.append(float(L))
        m, v = 0.9 * m + 0.1 * q.grad, 0.999 * v + 0.001 * q.grad ** 2
        th = th - lr * (m / (1 - 0.9 ** (k + 1))) / ((v / (1 - 0.999 ** (k + 1))).sqrt() + 1e-8)
    return np.array(loss), th


def _diffusion_exact(case, sigma0, T, dt):
    """The three-stage scheme, or the two-stage one (scheme 1), with zero flux at the ends."""
    s, N = _up(sigma0), case["nx"]
    sf = 2 * s[1:] * s[:-1] / (s[1:] + s[:-1])
    for _ in range(case["steps"]):
        K = T ** case["law"]
        F = 0.5 * (K[1:] + K[:-1]) / (3 * sf)
        lo, up = torch.zeros_like(T), torch.zeros_like(T)
        lo[1:], up[:-1] = F, F
        pre = dt * 4 * T ** 3 / (4 * T ** 3 + 1) * N * N
        U = _tri(-pre * lo, 1 + pre * (lo + up), -pre * up, T ** 4)
        if case["scheme"] == 1:
            T = U.clamp(min=0) ** 0.25
            continue
        f = torch.zeros(N + 1, dtype=F64, device=DEV)
        f[1:-1] = F * (U[1:] - U[:-1]) * N
        rhs = dt * (f[1:] - f[:-1]) * N + T ** 4 + T
        T = _root(torch.ones_like(T), torch.ones_like(T), rhs - T, T)
    return T, U


def exact(case, seed):
    rng, kind = _rng(seed), case["kind"]
    if kind in ("slab", "group", "reference"):
        law, eps, n = case.get("law", 3), case.get("eps", 1e-2), case.get("steps", 1)
        each = GROUP_EPS if kind == "group" else (eps,)
        data = [_slab_inputs(case["nx"], case["nv"], law, e, rng) for e in each]
        return [_slab_exact(d, law, 0.5 / case["nx"], e, n, kind == "reference") for d, e in zip(data, each)]
    if kind == "batch":
        if case["slabs"] > 60:              # minutes
            return None
        members = _members(case["slabs"], case["fp32"])
        sigma0, bL, bR, E, O, T = _batch_inputs(members, rng)
        E, O, T, oe, oo, ot, op = E.clone(), O.clone(), T.clone(), 0, 0, 0, 0
        for w in members:
            N, P = w.N, w.P
            e, o, t = E[oe:oe + N * P], O[oo:oo + (N + 1) * P], T[ot:ot + N]
            r = _slab_exact((w.mu, w.omega, sigma0[ot:ot + N], bL[op:op + P], bR[op:op + P], e.reshape(N, P),
                             o.reshape(N + 1, P), t), w.m, w.dt, w.eps, case["steps"])
            e.copy_(r[0].reshape(-1))
            o.copy_(r[1].reshape(-1))
            t.copy_(r[2])
            oe, oo, ot, op = oe + N * P, oo + (N + 1) * P, ot + N, op + P
        return E, O, T
    if kind == "plane":
        if case["nx"] * case["ny"] > 2500:  # dense matrices of every cell
            return None
        mu, eta, om, b, sigma0, *state = _plane_inputs(case, rng)
        S = _Plane(case, mu, eta, om, b, sigma0)
        for _ in range(case["steps"]):
            state = S.step(*state)
        return tuple(state)
    if kind in ("train", "predict"):
        rows, theta = _rows(case["rows"], rng), _theta(rng)
        norm = _norm(rows)
        if kind == "train":
            return _train_exact(theta, rows, norm, case["batch"], case["steps"])
        nm = _up(norm)
        return _net(_bf16(theta), (_up(rows)[:, :5] - nm[:5]) / nm[5:10])
    sigma0, T = _diffusion_inputs(case, rng)
    return _diffusion_exact(case, sigma0, _up(T), 2e-4)
