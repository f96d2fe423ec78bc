"""The workloads that this library is timed on.

Each case is one pass of a program that uses the library through its public
classes, with the sizes and parameters of the repository's own workloads (the
seeded suspensions, the 512-system ensemble and the paper's lattice arrays) or
generic ones around them. Kinds of pass:

  run       Simulator.run(steps, every): advance one suspension or an ensemble,
            record centres and mean positions, then read the state back
  step      Simulator.step(steps) and the state: a program that couples the
            swimmers to something else and looks at them after every step
  mobility  Simulator.mobility(X, F): one product for the caller's own forces
  averaged  StrokeAveraged.run(dt, steps) and the rates at the new state

listed() are the cases to watch, draw() gives others of the same ranges.
"""
import math

import numpy as np
import torch

import paper_1004_1932_amd as ad

DEVICE = "cuda:0" if torch.cuda.is_available() else "cpu"


class Params:
    """Model parameters of the seeded suspensions: a = eta = k = 1, ell = 4,
    lam = 1, T = 100, dt = 0.01."""
    a, eta, k, ell, lam, T, dt, steric_k, steric_r = 1.0, 1.0, 1.0, 4.0, 1.0, 100.0, 0.01, 0.0, 2.0


class StericParams(Params):
    """The same with the steric repulsion of the 65536-sphere suspension."""
    steric_k = 100.0


class ArrayParams(Params):
    """The aligned-pair parameters in SI units, which the array experiments
    use too: ell = 5 um, omega = 500 /s, lam = 0.1 ell, a = 0.2 ell."""
    ell = 5e-6
    a, eta, k, lam = 0.2 * ell, 1e-3, 1e-3, 0.1 * ell
    T = 2.0 * math.pi / 500.0
    dt = T / 5000


def listed():
    return [
        # the smallest suspension (8 dumbbells), a stretch of its run in plain
        # FP64, recorded ten times: the reference run people check others with
        case("n16 fp64", S=8, side=40.0, precision="fp64", steps=500, every=50),
        # 27 dumbbells stepped one call at a time by a program that reads the
        # state back after each step: launches and host work count
        case("27 dumbbells, step by step", kind="step", S=27, side=60.0, steps=1),
        # the 512-sphere suspension: too small to fill the chip
        case("n512", S=256, side=120.0, steps=100, every=50),
        # an odd size with Brownian noise and the paper's own integrator
        case("n1354 brownian heun", S=677, side=165.0, integrator="heun", kT=0.01, steps=100, every=50),
        # the headline suspension, RK4
        case("n4096", S=2048, side=240.0, steps=100, every=50),
        # the same in plain FP64, the sequential sum
        case("n4096 fp64", S=2048, side=240.0, precision="fp64", steps=10, every=10),
        # a larger one of odd size: enough pairs to fill the chip
        case("n15002", S=7501, side=370.0, steps=20, every=20),
        # the largest suspension, with steric contacts
        case("n65536 steric", S=32768, side=800.0, steric=True, steps=4, every=4),
        # 512 uneven systems of 16 to 400 dumbbells, dense, in one launch per stage
        case("512 systems", W=512, S=16, most=400, density=0.02, steps=10, every=10),
        # ten of the paper's largest arrays, with the tensor of its runs
        case("ten 7^3 arrays rpy", W=10, S=343, lattice=7, tensor="rpy", steps=50, every=25),
        # one velocity evaluation for forces that the caller computed
        case("mobility n6000 fp64", kind="mobility", S=3000, side=275.0, precision="fp64_tiled", tensor="rpy"),
        # the stroke-averaged equations of a 7^3 array over one period
        case("averaged 7^3", kind="averaged", S=343, lattice=7, steps=20),
    ]


def case(name, kind="run", S=8, side=0.0, W=1, most=0, density=0.0, lattice=0, precision="fp32c",
         integrator="rk4", tensor="oseen", kT=0.0, steric=False, steps=1, every=0):
    """S: dumbbells per system; W: systems; most: systems are uneven, of S to
    `most` dumbbells; lattice: cubic arrays of that many dumbbells a side."""
    c = dict(kind=kind, S=S, side=side, W=W, most=most, density=density, lattice=lattice, precision=precision,
             integrator=integrator, tensor=tensor, kT=kT, steric=steric, steps=steps, every=every)
    return dict(c, name=name) if name else c


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(("single", "single", "single", "fp64", "steric", "ensemble", "arrays", "mobility", "averaged"))
    integrator, kT = rng.choice((("rk4", 0.0), ("rk4", 0.0), ("heun", 0.0), ("heun", 0.01)))
    tensor = rng.choice(("oseen", "oseen", "rpy"))
    if kind == "single":
        S = _log(rng, 8, 16000)
        steps = rng.randrange(1, max(2, min(200, 100000000 // (S * S))))
        return case(None, S=S, side=18.0 * S ** (1 / 3), integrator=integrator, kT=kT, tensor=tensor, steps=steps,
                    every=rng.choice((steps, max(1, steps // 4))))
    if kind == "fp64":
        S = _log(rng, 8, 5000)
        return case(None, S=S, side=18.0 * S ** (1 / 3), precision=rng.choice(("fp64", "fp64", "fp64_tiled")),
                    integrator=integrator, tensor=tensor, steps=(4 if S > 500 else 50), every=2)
    if kind == "steric":
        S = _log(rng, 1000, 30000)
        return case(None, S=S, side=25.0 * S ** (1 / 3), steric=True, steps=2, every=2)
    if kind == "ensemble":
        most = rng.randrange(100, 401)
        return case(None, W=_log(rng, 16, 500), S=16, most=most, density=0.02, tensor=tensor, steps=4, every=4)
    if kind == "arrays":
        x = rng.randrange(3, 10)
        return case(None, W=_log(rng, 4, 64), S=x ** 3, lattice=x, integrator=integrator if kT == 0.0 else "rk4",
                    tensor=tensor, steps=8 if x > 6 else 40, every=8)
    if kind == "mobility":
        S = _log(rng, 20, 6000)
        return case(None, kind="mobility", S=S, side=18.0 * S ** (1 / 3),
                    precision=rng.choice(("fp64", "fp64_tiled")), tensor=tensor)
    S = _log(rng, 27, 2500)
    return case(None, kind="averaged", S=S, side=10 * ArrayParams.ell * S ** (1 / 3), steps=rng.choice((5, 20)))


# ---------------------------------------------------------------- inputs

def _params(c):
    if c["lattice"] or c["kind"] == "averaged":
        return ArrayParams
    return StericParams if c["steric"] else Params


def _sizes(c):
    """Dumbbells per system; uneven ones as in the 512-system ensemble, whose
    sizes are the same for every draw of the positions."""
    if c["most"]:
        return np.random.default_rng(0).integers(c["S"], c["most"] + 1, c["W"])
    return np.full(c["W"], c["S"])


def _unit(v):
    return v / np.linalg.norm(v, axis=-1, keepdims=True)


def _close(X, system, rmin, G):
    """Per sphere: whether another dumbbell's sphere of smaller index lies
    closer than rmin in the same system (cells of side rmin, G a side)."""
    X = torch.as_tensor(X, device=DEVICE)
    system = torch.as_tensor(system, device=DEVICE)
    n = X.shape[0]
    cell = torch.floor(X / rmin).to(torch.int64) + G // 2
    key = ((system * G + cell[:, 0]) * G + cell[:, 1]) * G + cell[:, 2]
    key, order = torch.sort(key, stable=True)
    x = X[order]
    hit = torch.zeros(n, dtype=torch.bool, device=DEVICE)
    for d in range(27):
        want = key + ((d // 9 - 1) * G + (d // 3 % 3 - 1)) * G + (d % 3 - 1)
        lo, hi = torch.searchsorted(key, want), torch.searchsorted(key, want, right=True)
        for k in range(int((hi - lo).max())):
            at = (lo + k).clamp(max=n - 1)
            near = ((x[at] - x) ** 2).sum(1) < rmin * rmin
            hit |= near & (lo + k < hi) & (order[at] // 2 < order // 2)
    out = torch.zeros_like(hit)
    out[order] = hit
    return out.cpu().numpy()


def _suspension(c, seed):
    """Positions (N, 3), phases (S,) and dumbbells per system: uniform centres
    in a cube, uniform axes and phases; a dumbbell that overlaps another one
    is drawn again. (With steric forces some pairs start in contact.)"""
    rng = np.random.default_rng(seed)
    p, S = _params(c), _sizes(c)
    n = int(S.sum())
    phi = rng.uniform(0.0, 2.0 * math.pi, n)
    L = (p.ell + p.lam * np.sin(phi))[:, None]
    if c["lattice"]:
        g = np.arange(c["lattice"])
        idx = np.stack(np.meshgrid(g, g, g, indexing="ij"), -1).reshape(-1, 3)
        R = 10 * p.ell * (np.tile(idx, (c["W"], 1, 1)) - 0.5 * (c["lattice"] - 1) + rng.uniform(-1, 1, (c["W"], 1, 3)))
        R, axis = R.reshape(-1, 3), _unit(rng.standard_normal((n, 3)))
    else:
        system = np.repeat(np.arange(len(S)), S)
        side = (2.0 * S / c["density"]) ** (1 / 3) if c["density"] else np.full(len(S), c["side"])
        side, rmin = side[system][:, None], p.a * (1.8 if c["steric"] else 2.0)
        G = int((side.max() + 2 * p.ell) / rmin) + 6
        R, axis = np.empty((n, 3)), np.empty((n, 3))
        again = np.arange(n)
        while len(again):
            R[again] = rng.uniform(-0.5, 0.5, (len(again), 3)) * side[again]
            axis[again] = _unit(rng.standard_normal((len(again), 3)))
            if c["kind"] == "averaged":
                break
            X = np.stack([R - 0.5 * L * axis, R + 0.5 * L * axis], 1).reshape(-1, 3)
            again = np.nonzero(_close(X, np.repeat(system, 2), rmin, G).reshape(-1, 2).any(1))[0]
    X = np.stack([R - 0.5 * L * axis, R + 0.5 * L * axis], 1).reshape(-1, 3)
    return X, phi, S, R, axis


def _centres(c, seed):
    """Centres, axes and phases for the stroke-averaged equations, which hold
    for separations of several lengths: a lattice, or a jittered one."""
    X, phi, S, R, axis = _suspension(c, seed)
    if not c["lattice"]:
        x = math.ceil(round(c["S"] ** (1 / 3), 6))
        g = np.arange(x)
        idx = np.stack(np.meshgrid(g, g, g, indexing="ij"), -1).reshape(-1, 3)[: c["S"]]
        rng = np.random.default_rng(seed + 1)
        R = 10 * ArrayParams.ell * (idx - 0.5 * (x - 1) + rng.uniform(-0.3, 0.3, idx.shape))
    return R, axis, phi


def _caller_forces(c, seed):
    """Force-free pairs, as swimmers' springs give, plus a weak drive."""
    f = np.random.default_rng(seed + 2).standard_normal((c["S"], 3))
    g = 0.1 * np.random.default_rng(seed + 3).standard_normal((2 * c["S"], 3))
    return np.stack([-f, f], 1).reshape(-1, 3) + g


def _on_gpu(v):
    return torch.as_tensor(np.ascontiguousarray(v), dtype=torch.float64).to(DEVICE)


def prepare(case, seed):
    c = case
    if c["kind"] == "averaged":
        R, N, phi = _centres(c, seed)
        return dict(c, sim=ad.StrokeAveraged(ArrayParams, _on_gpu(R), _on_gpu(N), _on_gpu(phi), device=DEVICE))
    X, phi, S, _, _ = _suspension(c, seed)
    if c["kind"] == "mobility":
        sim = ad.Simulator(_params(c), S, precision=c["precision"], device=DEVICE, launch="tuned", tensor=c["tensor"])
        return dict(c, sim=sim, X=_on_gpu(X), F=_on_gpu(_caller_forces(c, seed)))
    sim = ad.Simulator(_params(c), S, precision=c["precision"], integrator=c["integrator"], device=DEVICE,
                       launch="tuned", graph=True, tensor=c["tensor"], kT=c["kT"], seed=7)
    sim.set_state(_on_gpu(X), _on_gpu(phi))
    return dict(c, sim=sim)


def run(state):
    sim = state["sim"]
    if state["kind"] == "averaged":
        sim.run(ArrayParams.T / 20, state["steps"])
        dR, dN = sim.rhs()
        return {"R": sim.R, "N": sim.N, "dR": dR, "dN": dN}
    if state["kind"] == "mobility":
        return {"u": sim.mobility(state["X"], state["F"])}
    if state["kind"] == "step":
        sim.step(state["steps"])
        return {"X": sim.get_state()[0]}
    centres, com, _ = sim.run(state["steps"], state["every"])
    return {"X": sim.get_state()[0], "centres": centres, "com": com}


def _stages(c):
    return c["steps"] * (4 if c["integrator"] == "rk4" else 2)


def work(case):
    """Each ordered pair term once per stage (28 flops, 34 with the
    Rotne-Prager correction; about 90 for a stroke-averaged pair); the state,
    phases and records once."""
    c = case
    S = _sizes(c).astype(float)
    if c["kind"] == "averaged":
        return {"bytes": 8.0 * 19 * c["S"], "flops": 90.0 * c["S"] * (c["S"] - 1) * (4 * c["steps"] + 1)}
    pairs = float((2 * S * (2 * S - 1)).sum())
    term = 34.0 if c["tensor"] == "rpy" else 28.0
    if c["kind"] == "mobility":
        return {"bytes": float(144 * S.sum()), "flops": term * pairs}
    records = c["steps"] // c["every"] if c["every"] else 0
    return {"bytes": float(104 * S.sum() + records * (24 * S.sum() + 24 * len(S))), "flops": term * pairs * _stages(c)}


# ---------------------------------------------------------------- in 64 bits

def _velocity(p, X, F, rpy):
    """u = M(X) F for systems of equal size, X and F of shape (W, n, 3)."""
    W, n, _ = X.shape
    co, cr = 1.0 / (8.0 * math.pi * p.eta), p.a * p.a / (12.0 * math.pi * p.eta)
    u = F / (6.0 * math.pi * p.eta * p.a)
    rows = max(1, (1 << 24) // (W * n))
    for i0 in range(0, n, rows):
        i = torch.arange(i0, min(n, i0 + rows), device=X.device)
        r = [X[:, i, a, None] - X[:, None, :, a] for a in range(3)]
        r2 = r[0] * r[0] + r[1] * r[1] + r[2] * r[2]
        r2[:, i - i0, i] = math.inf
        ir = 1.0 / r2.sqrt()
        t = (r[0] * F[:, None, :, 0] + r[1] * F[:, None, :, 1] + r[2] * F[:, None, :, 2]) / r2
        for a in range(3):
            Fa = F[:, None, :, a]
            s = co * ir * (Fa + t * r[a])
            if rpy:
                s = s + cr * (ir / r2) * (Fa - 3.0 * t * r[a])
            u[:, i, a] += s.sum(-1)
    return u


def _steric(p, X):
    """Pairwise repulsion of one system, X of shape (1, n, 3)."""
    n = X.shape[1]
    F = torch.zeros_like(X)
    rows = max(1, (1 << 24) // n)
    for i0 in range(0, n, rows):
        i = torch.arange(i0, min(n, i0 + rows), device=X.device)
        r2 = sum((X[0, i, a, None] - X[0, None, :, a]) ** 2 for a in range(3))
        r2[i - i0, i] = math.inf
        at, j = torch.nonzero(r2 < p.steric_r ** 2, as_tuple=True)
        r = r2[at, j].sqrt()[:, None]
        F[0].index_add_(0, i[at], p.steric_k * (p.steric_r - r) / r * (X[0, i[at]] - X[0, j]))
    return F


def _forces(p, X, phi, t):
    L = p.ell + p.lam * torch.sin(2.0 * math.pi / p.T * t + phi)
    d = X[:, 1::2] - X[:, 0::2]
    r = d.square().sum(-1).sqrt()
    f = (-p.k * (r - L) / r)[..., None] * d
    F = torch.stack([-f, f], 2).reshape(X.shape)
    return F + _steric(p, X) if p.steric_k else F


def _normals(seed, spheres, step):
    """Three standard normals per sphere of one step: Philox4x32-10 with
    counter (sphere, step) and key seed, and Box-Muller."""
    low = np.uint64(0xFFFFFFFF)
    x = [spheres.astype(np.uint64), np.full(len(spheres), step, np.uint64), np.zeros(len(spheres), np.uint64),
         np.zeros(len(spheres), np.uint64)]
    k = [seed & 0xFFFFFFFF, seed >> 32]
    for _ in range(10):
        m0, m1 = x[0] * np.uint64(0xD2511F53), x[2] * np.uint64(0xCD9E8D57)
        x = [(m1 >> np.uint64(32)) ^ x[1] ^ np.uint64(k[0]), m1 & low,
             (m0 >> np.uint64(32)) ^ x[3] ^ np.uint64(k[1]), m0 & low]
        k = [(k[0] + 0x9E3779B9) & 0xFFFFFFFF, (k[1] + 0xBB67AE85) & 0xFFFFFFFF]
    u = [(v.astype(np.float64) + 0.5) / 2.0 ** 32 for v in x]
    r = [np.sqrt(-2.0 * np.log(u[0])), np.sqrt(-2.0 * np.log(u[2]))]
    return np.stack([r[0] * np.cos(2 * math.pi * u[1]), r[0] * np.sin(2 * math.pi * u[1]),
                     r[1] * np.cos(2 * math.pi * u[3])], -1)


def _advance(c, p, X, phi, sphere0):
    """(state, [(centres, mean position) per record]) of systems of one size."""
    rpy, dt, kept = c["tensor"] == "rpy", p.dt, []

    def u(Y, t):
        return _velocity(p, Y, _forces(p, Y, phi, t), rpy)

    for n in range(c["steps"]):
        t = n * dt
        k1 = u(X, t)
        if c["integrator"] == "rk4":
            k2 = u(X + 0.5 * dt * k1, t + 0.5 * dt)
            k3 = u(X + 0.5 * dt * k2, t + 0.5 * dt)
            k4 = u(X + dt * k3, t + dt)
            X = X + dt / 6.0 * (k1 + 2.0 * k2 + 2.0 * k3 + k4)
        else:
            xi = 0.0
            if c["kT"] > 0:
                at = (sphere0[:, None] + np.arange(X.shape[1])).reshape(-1)
                xi = _on_gpu(_normals(7, at, n)).reshape(X.shape)
                xi = math.sqrt(2.0 * c["kT"] * dt / (6.0 * math.pi * p.eta * p.a)) * xi
            X = X + 0.5 * dt * (k1 + u(X + dt * k1 + xi, t + dt)) + xi
        if c["every"] and (n + 1) % c["every"] == 0:
            kept.append((0.5 * (X[:, 0::2] + X[:, 1::2]), X.mean(1)))
    return X, kept


def _averaged_rates(R, N, phi):
    """dR/dt and dN/dt of the stroke-averaged far-field equations."""
    p = ArrayParams
    w, lr = 2.0 * math.pi / p.T, p.lam / p.ell
    D = R[:, None] - R[None]
    d = D.square().sum(-1)
    d.fill_diagonal_(math.inf)
    d = d.sqrt()
    e = D / d[..., None]
    s, r = (e * N[:, None]).sum(-1), (e * N[None]).sum(-1)
    q = (N[:, None] * N[None]).sum(-1)
    sn = torch.sin(phi[:, None] - phi[None])
    x = p.ell / d
    aN = 2 * s + 4 * q * r - 10 * s * r * r
    aD = 1 + 2 * q * q - 5 * s * s - 5 * r * r - 20 * q * s * r + 35 * s * s * r * r
    J = (p.a * w * 9 / 64 * lr * lr * sn * x ** 4)[..., None] * (N[:, None] * aN[..., None] + e * aD[..., None])
    b = 3 * s + 6 * r * q + 6 * s * q * q - 7 * s ** 3 - 21 * s * r * r - 42 * q * s * s * r + 63 * s ** 3 * r * r
    K = ((w * 15 / 64 * p.a / p.ell * lr * lr * sn * x ** 5 * b)[..., None] * e).sum(1)
    return J.sum(1), -(K - N * (N * K).sum(-1, keepdim=True))


def exact(case, seed):
    c, p = case, _params(case)
    if c["kind"] == "averaged":
        R, N, phi = (_on_gpu(v) for v in _centres(c, seed))
        h = p.T / 20
        for _ in range(c["steps"]):
            a = [_averaged_rates(R, N, phi)]
            for f in (0.5, 0.5, 1.0):
                a.append(_averaged_rates(R + f * h * a[-1][0], N + f * h * a[-1][1], phi))
            R, N = (v + h / 6 * (a[0][k] + 2 * a[1][k] + 2 * a[2][k] + a[3][k]) for k, v in ((0, R), (1, N)))
            N = N / N.square().sum(-1, keepdim=True).sqrt()
        dR, dN = _averaged_rates(R, N, phi)
        return {"R": R, "N": N, "dR": dR, "dN": dN}
    X, phi, S, _, _ = _suspension(c, seed)
    X, phi = _on_gpu(X), _on_gpu(phi)
    if c["kind"] == "mobility":
        F = _on_gpu(_caller_forces(c, seed))
        return {"u": _velocity(p, X[None], F[None], c["tensor"] == "rpy")[0]}
    first = np.concatenate([[0], np.cumsum(S)])
    records = c["steps"] // c["every"] if c["every"] else 0
    end = torch.empty_like(X)
    centres = X.new_empty((records, len(phi), 3))
    com = X.new_empty((records, len(S), 3))
    for size in sorted(set(S.tolist())):
        which = np.nonzero(S == size)[0]
        at = torch.as_tensor(first[which][:, None] + np.arange(size), device=X.device)
        both = (2 * at[..., None] + torch.arange(2, device=X.device)).reshape(len(which), -1)
        Y, kept = _advance(c, p, X[both], phi[at], 2 * first[which])
        end[both] = Y
        for k, (cen, mean) in enumerate(kept):
            centres[k, at] = cen
            com[k, torch.as_tensor(which, device=X.device)] = mean
    return {"X": end} if c["kind"] == "step" else {"X": end, "centres": centres, "com": com}
