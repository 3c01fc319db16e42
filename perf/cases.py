"""Performance cases of the framework: what its users run, over the sizes, storage types and options they run it with.

Three kinds of work:

``steps``  a time-marching program: ``nsteps`` lattice steps per call, then the two buffers change places.  Lattice,
           grid, storage type, path-length mode, walls (the lid-driven cavity) and the ES-BGK Prandtl number vary.
``log``    one step with the fused statistics and their read-back, as the alpha log takes them after every step.
``grad``   a training step: a checkpointed differentiable rollout with its accumulated dissipation loss and the
           final kinetic energy, and the gradients with respect to the initial state and the body force.

``exact`` is the same in double precision, written with plain torch operations.
"""
from __future__ import annotations

import math

import torch
from torch.utils.checkpoint import checkpoint

from paper_2203_12946_amd import adjoint
from paper_2203_12946_amd import eselbm

ITEM = {"f64": 8, "f32": 4, "f32s": 4, "f16s": 2}
KE_2D, KE_3D = 0.05, 0.1 / math.sqrt(3.0)  # vortex speeds of the repository's workloads


def _case(kind, D, n, dtype, nsteps, nu, mode="higher", walls=0, prandtl=1.0, force=False, diss=0.0, ckpt=0, name=None):
    nx, ny, nz = (tuple(n) + (1,))[:3]
    c = dict(kind=kind, D=D, nx=nx, ny=ny, nz=nz, dtype=dtype, nsteps=nsteps, nu=nu, mode=mode, walls=walls,
             prandtl=prandtl, force=force, diss=diss, ckpt=ckpt)
    return dict(c, name=name) if name else c


def _nu_tgv3d(nx):
    """Lattice viscosity of the Re 1600 Taylor-Green vortex with nx cells per period."""
    return KE_3D * (nx / (2 * math.pi)) / 1600.0


def listed():
    return [
        # the smallest workload, a 64 x 64 Taylor-Green vortex in double precision: launches and latency
        _case("steps", 2, (64, 64), "f64", 100, 0.01, name="tgv2d_64_f64"),
        # the same flow logged step by step, the smallest call there is
        _case("log", 2, (64, 64), "f64", 1, 0.01, name="alpha_log_64_f64"),
        # the doubly periodic 1024 x 1024 flow of the paper's shear-layer study: fits the last-level cache
        _case("steps", 2, (1024, 1024), "f32", 20, 1e-4, name="d2q9_1024_f32"),
        # the headline: the 256^3 Taylor-Green vortex at Re 1600, in the three widths of storage
        _case("steps", 3, (256, 256, 256), "f32", 20, _nu_tgv3d(256), name="tgv3d_256_f32"),
        _case("steps", 3, (256, 256, 256), "f64", 10, _nu_tgv3d(256), name="tgv3d_256_f64"),
        _case("steps", 3, (256, 256, 256), "f16s", 20, _nu_tgv3d(256), name="tgv3d_256_f16s"),
        # an ordinary box of odd extents in the format that meets the 1e-6 parity bar, an odd count of steps
        _case("steps", 3, (203, 97, 131), "f32s", 7, _nu_tgv3d(203), name="box_203x97x131_f32s"),
        # the lid-driven cavity, every axis walled
        _case("steps", 3, (192, 192, 192), "f32", 10, 0.05 * 192 / 1000, walls=7, name="cavity3d_192_f32"),
        # the entropic ES-BGK collision at the Prandtl number of air
        _case("steps", 3, (160, 160, 160), "f32", 5, _nu_tgv3d(160), prandtl=0.71, name="esbgk3d_160_f32"),
        # the iterative root search that the closed form is compared with, on a ragged box
        _case("steps", 3, (150, 150, 120), "f32", 5, _nu_tgv3d(150), mode="elbm", name="elbm3d_150_f32"),
        # training steps: the 2-D one, bound by launches, and the forced 3-D one with its dissipation loss
        _case("grad", 2, (256, 256), "f32", 50, 1e-4, ckpt=10, name="grad2d_256_f32"),
        _case("grad", 3, (128, 128, 128), "f32", 20, _nu_tgv3d(128), force=True, diss=_nu_tgv3d(128), ckpt=5,
              name="grad3d_128_f32"),
    ]


MOST_BYTES = 72e9  # of one pass: the listed 256^3 cases


def draw(rng):
    def size(lo, hi):
        return max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi + 1))))))

    kind = rng.choice(["steps"] * 6 + ["log", "grad", "grad"])
    D = rng.choice([2, 3])
    dtype = rng.choice(["f64", "f32", "f32", "f32s", "f16s"] if kind != "grad" else ["f64", "f32", "f32", "f32s"])
    base = size(32, 2048) if D == 2 else size(16, 256)
    if kind == "grad":
        base = min(base, 512 if D == 2 else 128)
    # sides of comparable length: half of the grids equal sides, half ragged
    n = [base] * D if rng.random() < 0.5 else [max(8, int(base * rng.uniform(0.5, 1.0))) for _ in range(D)]
    cells = math.prod(n)
    mode, walls, prandtl, force, diss, ckpt = "higher", 0, 1.0, False, 0.0, 0
    if kind == "steps":
        what = rng.choice(["plain", "plain", "plain", "walls", "esbgk", "mode"])
        if what == "walls":
            walls = rng.choice([(1 << D) - 1, 2])
        elif what == "esbgk":
            prandtl = rng.choice([0.71, 0.5, 1.4])
        elif what == "mode":
            mode = rng.choice(["bgk", "lower", "elbm", "iterate1"])
    nu = rng.uniform(0.5, 2.0) * (_nu_tgv3d(n[0]) if D == 3 else 0.01)
    if mode == "bgk":
        nu = max(nu, 0.01)  # alpha = 2 has no entropic stabilisation
    nsteps = 1 if kind == "log" else size(1, 100 if D == 2 else 20)
    if kind == "grad":
        nsteps = size(5, 60 if D == 2 else 20)
        ckpt = rng.randint(2, max(2, nsteps // 2))
        force = dtype == "f32" and rng.random() < 0.5
        diss = nu if rng.random() < 0.5 else 0.0
    q = 9 if D == 2 else 27
    per_step = 2 * q * ITEM[dtype] * cells * (4 if kind == "grad" else 1)
    nsteps = max(1, min(nsteps, int(MOST_BYTES / per_step)))
    return _case(kind, D, n, dtype, nsteps, nu, mode, walls, prandtl, force, diss, ckpt)


# ---------------------------------------------------------------------------------------------------------------
# Inputs
# ---------------------------------------------------------------------------------------------------------------
def _velocities(D):
    """Population i has velocity c_ia = (i / 3^a) mod 3 - 1, x fastest."""
    q = 9 if D == 2 else 27
    return [[(i // 3 ** a) % 3 - 1 for a in range(D)] for i in range(q)]


def _weights(D):
    return [math.prod(2.0 / 3.0 if v == 0 else 1.0 / 6.0 for v in c) for c in _velocities(D)]


def _factors(u):
    """Per-axis factors of the product-form entropic equilibrium, [axis][c + 1]."""
    out = []
    for ua in u:
        s = torch.sqrt(1.0 + 3.0 * ua * ua)
        out.append([(2 * s - 1) / 6 - ua / 2, 2 * (2 - s) / 3, (2 * s - 1) / 6 + ua / 2])
    return out


def _feq(D, rho, F, i):
    r = rho
    for a, v in enumerate(_velocities(D)[i]):
        r = r * F[a][v + 1]
    return r


def _fields(case, seed, dev):
    """Density [grid] and velocity components of a seeded flow: Taylor-Green vortices with random phases on a mean
    flow, plus noise; in the cavity a vortex that vanishes at the walls."""
    D = case["D"]
    shape = (case["ny"], case["nx"]) if D == 2 else (case["nz"], case["ny"], case["nx"])
    g = torch.Generator(device=dev).manual_seed(seed)
    r = torch.rand(8, generator=g, device=dev, dtype=torch.float64).tolist()
    walled = case["walls"] != 0
    xs = []
    for a in range(D):
        n = shape[D - 1 - a]
        t = (torch.arange(n, device=dev, dtype=torch.float64) + (0.5 if walled else 0.0)) / n
        t = math.pi * t if walled else 2 * math.pi * (t + r[a])
        xs.append(t.reshape([-1 if k == D - 1 - a else 1 for k in range(D)]))
    u0 = KE_2D if D == 2 else KE_3D
    one = torch.ones(shape, device=dev, dtype=torch.float64)
    if walled:
        u0 *= 0.5 + 0.5 * r[3]
        sz = 1.0 if D == 2 else torch.sin(xs[2]) ** 2
        u = [u0 * torch.sin(xs[0]) ** 2 * torch.sin(2 * xs[1]) * sz, -u0 * torch.sin(2 * xs[0]) * torch.sin(xs[1]) ** 2 * sz]
        rho = one.clone()
    else:
        cz = 1.0 if D == 2 else torch.cos(xs[2])
        u = [0.01 * r[4] + u0 * torch.sin(xs[0]) * torch.cos(xs[1]) * cz, 0.01 * r[5] - u0 * torch.cos(xs[0]) * torch.sin(xs[1]) * cz]
        p = torch.cos(2 * xs[0]) + torch.cos(2 * xs[1])
        rho = one + (0.75 * u0 * u0 * p if D == 2 else 3.0 * u0 * u0 / 16.0 * p * (torch.cos(2 * xs[2]) + 2.0))
    u += [0.0] * (D - len(u))
    u = [one * ua + 1e-4 * torch.randn(shape, generator=g, device=dev, dtype=torch.float64) for ua in u]
    F = None
    if case["force"]:
        F = (1e-6 * torch.randn((D,) + shape, generator=g, device=dev, dtype=torch.float64)).float()
    return rho, u, F


STORAGE = {"f64": torch.float64, "f32": torch.float32, "f32s": torch.float32, "f16s": torch.float16}


def _initial_state(case, rho, u):
    """The equilibrium of the fields in the storage type (f32s and f16s hold f - w)."""
    D = case["D"]
    w, F = _weights(D), _factors(u)
    f = torch.empty((len(w),) + rho.shape, device=rho.device, dtype=STORAGE[case["dtype"]])
    for i in range(len(w)):
        v = _feq(D, rho, F, i)
        f[i] = v - w[i] if case["dtype"].endswith("s") else v
    return f


LID = 0.05  # wall speed of the cavity


def prepare(case, seed):
    D = case["D"]
    shape = (case["ny"], case["nx"]) if D == 2 else (case["nz"], case["ny"], case["nx"])
    dev = torch.device("cuda", torch.cuda.current_device())
    rho, u, F = _fields(case, seed, dev)
    s = eselbm.Solver("D2Q9" if D == 2 else "D3Q27", shape, dtype=case["dtype"], mode=case["mode"])
    if case["walls"]:
        # the wall at the high end of the y axis is the lid
        s.set_walls([bool(case["walls"] >> a & 1) for a in range(D)], {(1, 1): (LID,) + (0.0,) * (D - 1)})
    if case["prandtl"] != 1.0:
        s.set_prandtl(case["prandtl"])
    f = _initial_state(case, rho, u)
    if case["kind"] == "grad":
        return dict(case=case, s=s, f=f.requires_grad_(True), F=F.requires_grad_(True) if F is not None else None)
    if case["kind"] == "log":
        s.set_stats(True)
    return dict(case=case, s=s, a=f, b=s.empty_state())


def run(state):
    case, s, tau = state["case"], state["s"], 3.0 * state["case"]["nu"]
    if case["kind"] == "grad":
        f, F = state["f"], state["F"]
        fN, diss = adjoint.rollout(s, f, tau, case["nsteps"], case["ckpt"], force=F, diss_weight=case["diss"] or None)
        loss = adjoint.kinetic_energy(s, fN)
        if case["diss"]:
            loss = loss + diss
        wrt = [f] if F is None else [f, F]
        grads = torch.autograd.grad(loss, wrt)
        return {"state": fN.detach(), "grad_state": grads[0], "grad_force": grads[1] if F is not None else None,
                "loss": loss.detach().to(f.dtype)}
    s.step(state["a"], state["b"], case["nsteps"], tau)
    state["a"], state["b"] = state["b"], state["a"]
    if case["kind"] == "log":
        st = s.stats(with_H=True)
        out = {k: st[k] for k in ("n_cells", "n_nonpos")}
        if case["dtype"] == "f64":
            out.update({k: st[k] for k in ("mass", "kinetic", "H", "alpha_min", "alpha_max", "alpha_mean")})
        return dict(out, state=state["a"])
    return state["a"]


def work(case):
    """Each population read and written once a step; a gradient step moves the state forward (f read and written),
    and back (f and the adjoint read, the adjoint written)."""
    q = 9 if case["D"] == 2 else 27
    cells, item = case["nx"] * case["ny"] * case["nz"], ITEM[case["dtype"]]
    # per cell update: moments, equilibrium, departures x and their power sums, relaxation: about 25 operations a
    # population; the adjoint about twice that
    b, fl = 2 * q * item, 25 * q
    if case["kind"] == "grad":
        b, fl = b + 3 * q * item, 3 * fl
        if case["force"]:
            b += 4 * case["D"] * 4
    return {"bytes": float(b) * cells * case["nsteps"], "flops": float(fl) * cells * case["nsteps"]}


# ---------------------------------------------------------------------------------------------------------------
# The same in double precision, with plain torch operations
# ---------------------------------------------------------------------------------------------------------------
def _root(a, b, c):
    return 2 * c / (b + torch.sqrt(b * b - 4 * a * c))


def _alpha(g, d, beta, mode):
    """Path length per cell from the lists of populations g and departures d = feq - g."""
    if mode == "bgk":
        return torch.full_like(g[0], 2.0)
    xmax = torch.zeros_like(g[0])
    with torch.no_grad():
        for gi, di in zip(g, d):
            xmax = torch.maximum(xmax, (di / gi).abs())
        gated = xmax < 1e-3
        # where the gate holds, departures of a fixed pattern stand in, so that no 0/0 arises
        patt = [0.01 * ((i % 3) - 1) for i in range(len(g))]
    x = [torch.where(gated, torch.full_like(gi, p), di / gi) for gi, di, p in zip(g, d, patt)]
    zero = torch.zeros_like(g[0])
    S2, C1, C, xmin = zero, zero, zero, zero
    M = {3: zero, 4: zero, 5: zero, 6: zero}
    for gi, xi in zip(g, x):
        gx2 = gi * xi * xi
        S2 = S2 + gx2
        C1 = C1 + 2 * gx2 / (2 + xi)
        C = C + gx2 * (60 + 60 * xi + 11 * xi * xi) / (60 + 90 * xi + 36 * xi * xi + 3 * xi ** 3)
        xn = torch.clamp(xi, max=0.0)
        t = gi * xn * xn
        for k in (3, 4, 5, 6):
            t = t * xn
            M[k] = M[k] + t
        xmin = torch.minimum(xmin, xi)
    b1 = 0.5 * S2
    aL = _root(0.5 * M[3], b1, C1)
    if mode == "higher":
        Bp = zero
        for gi, xi in zip(g, x):
            xp = torch.clamp(xi, min=0.0)
            y = aL * xp
            Bp = Bp + gi * xp ** 3 * (80 + 80 * y + 19 * y * y) / (64 + 96 * y + 44 * y * y + 6 * y ** 3)
        b = b1 - (2.0 / 15.0) * aL * beta * beta * Bp
        h = _root(beta * beta * M[3] / 6, b, C)
        hb = h * beta
        a = beta * beta * (M[3] / 6 - hb * M[4] / 12 + hb * hb * M[5] / 20 - hb ** 3 * M[6] / 5)
        al = _root(a, b, C)
    elif mode == "lower":
        al = aL
    else:
        al = _mirror(g, x, aL, -1.0 / xmin, full=mode == "elbm")
    amax = -1.0 / (beta * torch.clamp(xmin, max=-1e-300))
    al = torch.where((xmin < 0) & (al > amax), 0.5 * (1 + amax), al)
    return torch.where(gated, torch.full_like(al, 2.0), al)


def _mirror(g, x, aL, astar, full):
    """The root of H[f + a (feq - f)] = H[f] on (1, astar), or one Newton step towards it."""
    S = sum(gi * xi * torch.log1p(xi) for gi, xi in zip(g, x))
    lo, hi = torch.ones_like(aL), astar.clone()
    ok0 = (aL > lo) & (aL < hi)
    a = torch.where(ok0, aL, 0.5 * (lo + hi))
    seen = torch.zeros_like(ok0)
    for _ in range(12 if full else 1):
        Fv, Fp = -a * S, -S
        for gi, xi in zip(g, x):
            y = a * xi
            l1 = torch.log1p(y)
            # (1 + y) log(1 + y) - y without its cancellation for small y
            ser = sum((-1.0) ** k * y ** k / (k * (k - 1.0)) for k in range(2, 11))
            Fv = Fv + gi * torch.where(y.abs() < 0.01, ser, (1 + y) * l1 - y)
            Fp = Fp + gi * xi * l1
        if not full:
            an = a - Fv / Fp
            return torch.where(ok0 & (an > 1) & (an < astar), an, aL)
        seen = seen | (Fv > 0)
        hi = torch.where(Fv > 0, a, hi)
        lo = torch.where(Fv > 0, lo, a)
        an = a - Fv / Fp
        step = (an - a).abs() <= 1e-9 * an.abs()
        a = torch.where((an >= lo) & (an <= hi), an, 0.5 * (lo + hi))
        seen = seen | (step & (a < astar * (1 - 1e-6)))
    return torch.where(seen, a, aL)


def _quasi_equilibrium(D, feq, d, cpr):
    """feq exp(delta . phi) with the moments of feq and c_Pr times the stress, by Newton's method."""
    c = _velocities(D)
    pairs = [(a, b) for a in range(D) for b in range(a, D)]
    phi = [[1.0] + [float(v) for v in ci] + [float(ci[a] * ci[b]) for a, b in pairs] for ci in c]
    K, Q = len(phi[0]), len(c)
    tgt = [torch.zeros_like(feq[0]) for _ in range(K)]
    for k in range(1 + D, K):
        tgt[k] = -cpr * sum(d[i] * phi[i][k] for i in range(Q) if phi[i][k])
    delta = [torch.zeros_like(feq[0]) for _ in range(K)]

    def dot(i):
        return sum(delta[k] * phi[i][k] for k in range(K) if phi[i][k])

    for _ in range(6):
        J = [[torch.zeros_like(feq[0]) for _ in range(k + 1)] for k in range(K)]
        F = [t.clone() for t in tgt]
        for i in range(Q):
            r = feq[i] * torch.expm1(dot(i))
            for k in range(K):
                if not phi[i][k]:
                    continue
                F[k] -= r * phi[i][k]
                for m in range(k + 1):
                    if phi[i][m]:
                        J[k][m] += (feq[i] + r) * (phi[i][k] * phi[i][m])
        for j in range(K):  # Cholesky, then the two triangular solves
            J[j][j] = torch.sqrt(J[j][j] - sum((J[j][q] ** 2 for q in range(j)), torch.zeros_like(feq[0])))
            for r in range(j + 1, K):
                J[r][j] = (J[r][j] - sum((J[r][q] * J[j][q] for q in range(j)), torch.zeros_like(feq[0]))) / J[j][j]
        for k in range(K):
            for q in range(k):
                F[k] = F[k] - J[k][q] * F[q]
            F[k] = F[k] / J[k][k]
        for k in range(K - 1, -1, -1):
            for q in range(k + 1, K):
                F[k] = F[k] - J[q][k] * F[q]
            F[k] = F[k] / J[k][k]
            delta[k] = delta[k] + F[k]
    return [feq[i] * torch.expm1(dot(i)) for i in range(Q)]


def _pull(case, f):
    """Streaming: population i of a cell comes from the cell at - c_i; beyond a wall, from the wall's equilibrium
    with the mass that went into the walls."""
    D, walls = case["D"], case["walls"]
    c = _velocities(D)
    g = [torch.roll(f[i], tuple(c[i]), tuple(D - 1 - a for a in range(D))) for i in range(len(c))]
    if not walls:
        return g
    shape = f[0].shape
    w = _weights(D)
    out, inc, parts = torch.zeros_like(f[0]), torch.zeros_like(f[0]), []
    for i, ci in enumerate(c):
        taken = torch.zeros(shape, dtype=torch.bool, device=f[0].device)
        emit = torch.zeros_like(f[0])
        for a in range(D):
            if not (walls >> a & 1) or ci[a] == 0:
                continue
            side = 0 if ci[a] > 0 else 1
            uw = [LID if (a, side, b) == (1, 1, 0) else 0.0 for b in range(D)]
            e = float(_feq(D, torch.tensor(1.0, dtype=torch.float64),
                           _factors([torch.tensor(v, dtype=torch.float64) for v in uw]), i))
            m = torch.zeros(shape, dtype=torch.bool, device=f[0].device)
            m.select(D - 1 - a, 0 if side == 0 else shape[D - 1 - a] - 1).fill_(True)
            emit = torch.where(m & ~taken, torch.full_like(emit, e), emit)
            taken = taken | m
        out = out + torch.where(taken, f[len(c) - 1 - i] - w[i], torch.zeros_like(out))
        inc = inc + torch.where(taken, emit - w[i], torch.zeros_like(inc))
        parts.append((taken, emit))
    base = sum(torch.where(t, torch.full_like(out, w[i]), torch.zeros_like(out)) for i, (t, _) in enumerate(parts))
    rw = (base + out) / torch.where(base > 0, base + inc, torch.ones_like(base))
    return [torch.where(t, rw * e, gi) for (t, e), gi in zip(parts, g)]


def _step64(case, f, F=None):
    """One step of the list of populations f; returns the new list, with density, velocity and path length."""
    D, beta = case["D"], 1.0 / (6.0 * case["nu"] + 1.0)
    c = _velocities(D)
    g = _pull(case, f)
    rho = sum(g)
    u = [sum(g[i] * c[i][a] for i in range(len(c)) if c[i][a]) / rho for a in range(D)]
    Fu = _factors(u)
    feq = [_feq(D, rho, Fu, i) for i in range(len(c))]
    d = [e - gi for e, gi in zip(feq, g)]
    if case["prandtl"] != 1.0:
        pr, tau = case["prandtl"], 3.0 * case["nu"]
        extra = _quasi_equilibrium(D, feq, d, (1.0 - 1.0 / pr) / (1.0 + 1.0 / (2.0 * tau * pr)))
        d = [di + e for di, e in zip(d, extra)]
    del feq
    al = _alpha(g, d, beta, case["mode"])
    out = [gi + al * beta * di for gi, di in zip(g, d)]
    if F is not None:
        Ff = _factors([ua + F[a] / rho for a, ua in enumerate(u)])
        out = [o + _feq(D, rho, Ff, i) - _feq(D, rho, Fu, i) for i, o in enumerate(out)]
    return out, rho, u, al


def _moments64(D, f, F=None):
    c = _velocities(D)
    rho = sum(f)
    j = [sum(f[i] * c[i][a] for i in range(len(c)) if c[i][a]) for a in range(D)]
    return rho, [(ja + (0.5 * F[a] if F is not None else 0.0)) / rho for a, ja in enumerate(j)]


def _dissipation(D, u):
    """sum |curl u|^2 with periodic central differences."""
    def diff(v, a):
        return 0.5 * (torch.roll(v, -1, D - 1 - a) - torch.roll(v, 1, D - 1 - a))

    t = 0.0
    for a, b in ([(0, 1)] if D == 2 else [(1, 2), (2, 0), (0, 1)]):
        t = t + ((diff(u[b], a) - diff(u[a], b)) ** 2).sum()
    return t


def exact(case, seed):
    D = case["D"]
    dev = torch.device("cuda", torch.cuda.current_device())
    rho, u, F = _fields(case, seed, dev)
    f0 = _initial_state(case, rho, u).double()
    w = _weights(D)
    if case["dtype"].endswith("s"):
        for i in range(len(w)):
            f0[i] += w[i]
    shift = w if case["dtype"].endswith("s") else [0.0] * len(w)

    def stored(f):
        return torch.stack([fi - wi for fi, wi in zip(f, shift)])

    if case["kind"] == "grad":
        f0.requires_grad_(True)
        wrt = [f0]
        if F is not None:
            F = F.double().requires_grad_(True)
            wrt.append(F)

        def one(x, force):
            out = _step64(case, list(x.unbind(0)), force)[0]
            return torch.stack(out)

        x, loss = f0, 0.0
        for _ in range(case["nsteps"]):
            x = checkpoint(one, x, F, use_reentrant=False)
            if case["diss"]:
                loss = loss + case["diss"] * checkpoint(
                    lambda y, force: _dissipation(D, _moments64(D, list(y.unbind(0)), force)[1]), x, F, use_reentrant=False)
        r, v = _moments64(D, list(x.unbind(0)))
        loss = loss + 0.5 * (r * sum(va * va for va in v)).sum()
        grads = torch.autograd.grad(loss, wrt)
        return {"state": stored(x.detach().unbind(0)), "grad_state": grads[0], "grad_force": grads[1] if F is not None else None,
                "loss": loss.detach()}
    with torch.no_grad():
        f = list(f0.unbind(0))
        del f0, u
        for _ in range(case["nsteps"]):
            f, rho, v, al = _step64(case, f)
        if case["kind"] == "log":
            out = {"n_cells": None, "n_nonpos": None, "state": stored(f)}
            if case["dtype"] == "f64":
                H = sum((fi * (torch.log(fi / wi) - 1.0)).sum() for fi, wi in zip(f, w))
                out.update(mass=rho.sum(), kinetic=0.5 * (rho * sum(va * va for va in v)).sum(), H=H,
                           alpha_min=al.min(), alpha_max=al.max(), alpha_mean=al.mean())
            return out
        return stored(f)
