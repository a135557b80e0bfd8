"""Timing cases of the thin-film framework: the calls its users make, over the sizes, models
and options they make them with.

    newton    Grid.newton_iteration: one ADI-Newton iteration of one film (residual, y sweep,
              x sweep, update); every time step of every program is a few of these
    advance   Grid.advance: whole time steps with their Newton loop and step control
    ensemble  Ensemble.step: many films of different sizes stepped in lockstep
    rollout   adjoint.rollout and its backward pass: a gradient in the initial film and kappa
    penta     penta_solve: a batch of pentadiagonal systems on stored bands
    spectrum  radial_spectrum: the radial Fourier transform of a film

listed() and draw() give cases (dicts of plain values), prepare() a program's state before the
call, run() one call, work() the bytes and operations the path cannot do without and exact() the
same results from plain torch and numpy in 64 bits. Everything is float64, the framework's only
data type.
"""
import math

import numpy as np
import torch

from paper_1806_10550_amd import lib
from paper_1806_10550_amd.adjoint import rollout

DEV = "cuda:0"

# Film models: mean thickness, cell side (a 32nd of the most unstable wavelength, as in the
# benchmark films) and the step at which that film's fastest mode grows by the benchmark's amount.
MODELS = {
    "power": {"h0": 1.0, "ds": 0.67347, "dt": 0.2},
    "nlc": {"h0": 0.5, "ds": 2.0 * math.pi / 1.48212 / 32.0, "dt": 0.028},
    "polymer": {"h0": 3.9, "ds": 2.0 * math.pi / 1.55987 / 32.0, "dt": 7.1e-4},
}
KAPPA, B = 10.0, 0.1
ENS_SIZES = (256, 384, 512, 768, 1024)
NEWTON_PER_STEP = 6  # typical Newton iterations of one accepted step (work estimates only)


# ---- the cases ---------------------------------------------------------------------------

def listed():
    return [
        # the smallest film of the benchmark: launches and latency decide
        {"name": "newton_128", "path": "newton", "nx": 128, "ny": 128, "model": "power", "theta": 1.0},
        # an ordinary film (the adjoint workload's size)
        {"name": "newton_512", "path": "newton", "nx": 512, "ny": 512, "model": "power", "theta": 1.0},
        # the dewetting study's film: liquid crystal model, odd size, trapezoidal rule
        {"name": "newton_1637_nlc", "path": "newton", "nx": 1637, "ny": 1637, "model": "nlc", "theta": 0.5},
        # the spinodal / nucleation films
        {"name": "newton_2048", "path": "newton", "nx": 2048, "ny": 2048, "model": "power", "theta": 1.0},
        # a ragged rectangular polymer film: long rows, fewer of them
        {"name": "newton_3001x700_polymer", "path": "newton", "nx": 3001, "ny": 700, "model": "polymer", "theta": 1.0},
        # the throughput film
        {"name": "newton_8192", "path": "newton", "nx": 8192, "ny": 8192, "model": "power", "theta": 1.0},
        # a short run of the small film with fixed dt
        {"name": "advance_128", "path": "advance", "nx": 128, "ny": 128, "steps": 20, "adaptive": False, "mass": False},
        # the spinodal film's adaptive run, mass recorded at every step
        {"name": "advance_2048_adaptive", "path": "advance", "nx": 2048, "ny": 2048, "steps": 3, "adaptive": True,
         "mass": True},
        # a part of the film ensemble
        {"name": "ensemble_24", "path": "ensemble", "films": 24, "steps": 2},
        # forward and backward of the differentiable rollout at the adjoint workload's size
        {"name": "rollout_512", "path": "rollout", "n": 512, "steps": 10, "theta": 1.0},
        # stored-band solves of an ordinary odd shape
        {"name": "penta_777x1000", "path": "penta", "n": 777, "nlines": 1000, "transposed": False},
        # the evolving film's analysis at a size of the dewetting study
        {"name": "spectrum_2674", "path": "spectrum", "n": 2674, "periods": 40.0},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    x = rng.random()
    if x < 0.45:
        nx = _log_int(rng, 64, 8192)
        ny = _log_int(rng, 64, 8192)
        return {"path": "newton", "nx": nx, "ny": ny, "model": rng.choice(["power", "power", "nlc", "polymer"]),
                "theta": rng.choice([1.0, 0.5])}
    if x < 0.60:
        adaptive = rng.random() < 0.5
        nx, ny = _log_int(rng, 48, 1200), _log_int(rng, 48, 1200)
        return {"path": "advance", "nx": nx, "ny": ny, "steps": rng.randint(3, 12), "adaptive": adaptive,
                "mass": rng.random() < 0.5}
    if x < 0.70:
        return {"path": "ensemble", "films": rng.randint(4, 24), "steps": rng.randint(1, 2)}
    if x < 0.78:
        return {"path": "rollout", "n": _log_int(rng, 64, 512), "steps": rng.randint(4, 10),
                "theta": rng.choice([1.0, 0.5])}
    if x < 0.90:
        return {"path": "penta", "n": _log_int(rng, 64, 4096), "nlines": _log_int(rng, 16, 4096),
                "transposed": rng.random() < 0.5}
    return {"path": "spectrum", "n": _log_int(rng, 256, 2674), "periods": float(rng.choice([10, 20, 40]))}


# ---- inputs ------------------------------------------------------------------------------

def _gen(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed))
    return g


def _noise(g, *shape):
    return torch.rand(*shape, generator=g, device=DEV, dtype=torch.float64) * 2.0 - 1.0


def _film(g, ny, nx, h0):
    """h0 (1 + 0.01 U[-1, 1]), the benchmark films' initial noise."""
    return h0 * (1.0 + 0.01 * _noise(g, ny, nx))


def _set_model(grid, model):
    if model == "power":
        grid.set_model(KAPPA, B, 3, 2)
    else:
        getattr(grid, "set_model_" + model)()


def _newton_inputs(case, seed):
    g = _gen(seed)
    un = _film(g, case["ny"], case["nx"], MODELS[case["model"]]["h0"])
    uk = un * (1.0 + 1e-4 * _noise(g, case["ny"], case["nx"]))  # an iterate on its way
    return un, uk


def _advance_scheme(case):
    if case["adaptive"]:
        return dict(tol=1e-10, max_newton=10, adaptive=1, dt_min=1e-6, dt_max=1.0)
    return dict(tol=1e-10)


def _ensemble_films(case, seed):
    rng = np.random.default_rng(seed)
    qm = [math.sqrt(k * 0.017 / 2.0) for k in rng.uniform(5.0, 20.0, case["films"])]
    # every size in turn, so that the work depends on the number of films and not on the seed
    n = [ENS_SIZES[f % len(ENS_SIZES)] for f in range(case["films"])]
    kappa = [2.0 * q * q / 0.017 for q in qm]
    ds = [8.0 * 2.0 * math.pi / q / m for q, m in zip(qm, n)]
    dt = [0.5 * d ** 4 for d in ds]  # about the step the adaptive control settles at
    return n, kappa, ds, dt


def _rollout_inputs(case, seed):
    g = _gen(seed)
    n = case["n"]
    base = _film(g, n, n, 1.0)
    p0 = 1e-3 * _noise(g, n, n)
    target = _film(g, n, n, 1.0)
    return base, p0, target


def _penta_inputs(case, seed):
    """Bands like those of I + c J on a film: a fourth difference of strength k per cell."""
    g = _gen(seed)
    n, nl = case["n"], case["nlines"]
    k = 0.5 * (1.0 + 0.5 * _noise(g, n, nl))
    e = 0.05 * _noise(g, 2, n, nl)
    bands = torch.stack([k, -4.0 * k + e[0], 1.0 + 6.0 * k, -4.0 * k + e[1], k])
    bands[0, :2] = 0.0
    bands[1, :1] = 0.0
    bands[3, n - 1:] = 0.0
    bands[4, n - 2:] = 0.0
    return bands.contiguous(), _noise(g, n, nl)


def _spectrum_inputs(case, seed):
    """A film with waves of about the most unstable length over noise."""
    g = _gen(seed)
    n, P = case["n"], case["periods"]
    x = (torch.arange(n, device=DEV, dtype=torch.float64) + 0.5) / n
    h = 0.05 * (1.0 + 0.01 * _noise(g, n, n))
    a = _noise(g, 8)
    for i in range(4):
        kx, ky = P * math.cos(0.3 + i), P * math.sin(0.3 + i)
        h += 5e-4 * a[i] * torch.cos(2.0 * math.pi * (round(kx) * x[None, :] + round(ky) * x[:, None]) + a[4 + i])
    ds = 0.01
    return h.contiguous(), ds, 0.05, 5.0 * 2.0 * math.pi * P / (n * ds)


def prepare(case, seed):
    path = case["path"]
    if path == "newton":
        m = MODELS[case["model"]]
        un, uk = _newton_inputs(case, seed)
        grid = lib.Grid(case["nx"], case["ny"], m["ds"])
        _set_model(grid, case["model"])
        grid.set_scheme(theta=case["theta"])
        return {"path": path, "grid": grid, "un": un, "uk": uk, "out": torch.empty_like(un), "dt": m["dt"]}
    if path == "advance":
        h0 = _film(_gen(seed), case["ny"], case["nx"], 1.0)
        grid = lib.Grid(case["nx"], case["ny"], MODELS["power"]["ds"])
        grid.set_model(KAPPA, B, 3, 2)
        grid.set_scheme(**_advance_scheme(case))
        grid.set_diagnostics(case["mass"])
        return {"path": path, "grid": grid, "h0": h0, "h": h0.clone(), "steps": case["steps"], "dt": 0.1,
                "mass": case["mass"]}
    if path == "ensemble":
        n, kappa, ds, dt = _ensemble_films(case, seed)
        ens = lib.Ensemble(n, n, ds, kappa)
        ens.set_scheme(tol=1e-10, max_newton=10, adaptive=1, dt_min=1e-9, dt_max=1.0)
        packed0 = 1.0 + 0.01 * _noise(_gen(seed), ens.size)
        return {"path": path, "ens": ens, "packed0": packed0, "packed": packed0.clone(), "dt": dt,
                "steps": case["steps"]}
    if path == "rollout":
        base, p0, target = _rollout_inputs(case, seed)
        return {"path": path, "base": base, "p0": p0, "target": target, "steps": case["steps"],
                "theta": case["theta"], "kappa": torch.tensor(KAPPA, dtype=torch.float64, device=DEV)}
    if path == "penta":
        bands, rhs = _penta_inputs(case, seed)
        lib.load_shipped_tuning()
        return {"path": path, "bands": bands, "rhs": rhs, "x": torch.empty_like(rhs),
                "transposed": case["transposed"]}
    h, ds, h0, qmax = _spectrum_inputs(case, seed)
    return {"path": path, "h": h, "ds": ds, "h0": h0, "qmax": qmax}


def run(s):
    path = s["path"]
    if path == "newton":
        e, r, flags = s["grid"].newton_iteration(s["un"], s["uk"], s["out"], s["dt"])
        return {"u": s["out"], "e": e, "r": r, "flags": flags}
    if path == "advance":
        g, h = s["grid"], s["h"]
        h.copy_(s["h0"])
        g.bind(h)
        dt, log = g.advance(s["steps"], s["dt"], log=s["mass"])
        out = {"h": h, "dt": dt}
        if s["mass"]:
            out["mass"] = [x["mass"] for x in log]
            out["hmin"] = [x["hmin"] for x in log]
        return out
    if path == "ensemble":
        s["packed"].copy_(s["packed0"])
        s["ens"].bind(s["packed"])
        status, dts, statuses, _ = s["ens"].step(s["steps"], s["dt"])
        return {"h": s["packed"], "dt": np.array(dts), "status": np.array([status] + statuses)}
    if path == "rollout":
        p0 = s["p0"].detach().requires_grad_()
        kappa = s["kappa"].detach().requires_grad_()
        h = rollout(p0, kappa, s["base"], s["steps"], 0.1, MODELS["power"]["ds"], tol=1e-10, adj_tol=1e-10,
                    theta=s["theta"])
        loss = 0.5 * (h - s["target"]).square().sum()
        loss.backward()
        return {"h": h.detach(), "loss": loss.detach(), "grad_p0": p0.grad, "grad_kappa": kappa.grad}
    if path == "penta":
        return lib.penta_solve(s["bands"], s["rhs"], s["x"], transposed=s["transposed"])
    q, mean, count = lib.radial_spectrum(s["h"], s["ds"], s["h0"], 1.0, s["qmax"])
    return {"q": q, "mean": mean, "count": count}


def work(case):
    """Bytes: every input and output once. Operations: the assembly, one elimination and one
    back-substitution per sweep and cell (about 250) of each Newton iteration."""
    path = case["path"]
    if path == "newton":
        n = case["nx"] * case["ny"]
        return {"bytes": 24.0 * n, "flops": 250.0 * n}
    if path == "advance":
        n = case["nx"] * case["ny"] * case["steps"] * NEWTON_PER_STEP
        return {"bytes": 24.0 * n, "flops": 250.0 * n}
    if path == "ensemble":
        n = sum(ENS_SIZES[f % len(ENS_SIZES)] ** 2 for f in range(case["films"])) * case["steps"] * NEWTON_PER_STEP
        return {"bytes": 24.0 * n, "flops": 250.0 * n}
    if path == "rollout":  # forward, recomputation and the adjoint's iterations
        n = case["n"] ** 2 * case["steps"] * NEWTON_PER_STEP * 3
        return {"bytes": 24.0 * n, "flops": 250.0 * n}
    if path == "penta":
        n = case["n"] * case["nlines"]
        return {"bytes": 56.0 * n, "flops": 25.0 * n}
    n = case["n"] ** 2
    return {"bytes": 8.0 * n, "flops": 2.5 * n * math.log2(n)}


# ---- the same results in plain torch and numpy, 64 bits, on the CPU ------------------------
# Flux-form discretisation with even-reflection ghosts, D = flux differences of
# A grad(lap u) + B grad u with face means A, B of f0, f1; bands of I + c J_x and I + c J_y.

def _coeffs(model, h, kappa=KAPPA):
    """f0, f0', f1, f1'."""
    if model == "power":
        n, m = 3.0, 2.0
        f1 = kappa * h ** 3 * (-n * B ** n / h ** (n + 1) + m * B ** m / h ** (m + 1))
        f1p = kappa * (n * (n - 2) * B ** n * h ** (1 - n) - m * (m - 2) * B ** m * h ** (1 - m))
        return h ** 3, 3.0 * h ** 2, f1, f1p
    if model == "nlc":
        C, K, N, beta, w, b = 0.0857, 36.0, 1.67, 1.0, 0.05, 0.01
        z = (h - 2.0 * b) / w
        t = torch.tanh(z)
        g, gp, gpp = 0.5 * (1.0 + t), 0.5 * (1.0 - t * t) / w, -t * (1.0 - t * t) / w ** 2
        den = h * h + beta ** 2
        s, sp, spp = h / den, (beta ** 2 - h * h) / den ** 2, 2.0 * h * (h * h - 3.0 * beta ** 2) / den ** 3
        q, qp, qpp = g * s, gp * s + g * sp, gpp * s + 2.0 * gp * sp + g * spp
        p1 = K * (-3.0 * b ** 3 / h ** 4 + 2.0 * b ** 2 / h ** 3) + N * q * qp
        p2 = K * (12.0 * b ** 3 / h ** 5 - 6.0 * b ** 2 / h ** 4) + N * (qp * qp + q * qpp)
    else:
        C, Cst, Aox, Asi, d = 0.00581, 1.181, 41.25, -243.75, 191.0
        a2, c2 = Aox / (6.0 * math.pi), (Aox - Asi) / (6.0 * math.pi)
        p1 = -72.0 * Cst * h ** -10 + 3.0 * a2 * h ** -4 - 3.0 * c2 * (h + d) ** -4
        p2 = 720.0 * Cst * h ** -11 - 12.0 * a2 * h ** -5 + 12.0 * c2 * (h + d) ** -5
    return C * h ** 3, 3.0 * C * h ** 2, h ** 3 * p1, 3.0 * h ** 2 * p1 + h ** 3 * p2


def _lap(u, ds):
    e = torch.cat([u[:, :1], u, u[:, -1:]], 1)
    n = torch.cat([u[:1], u, u[-1:]], 0)
    return (e[:, 2:] + e[:, :-2] + n[2:] + n[:-2] - 4.0 * u) / ds ** 2


def _flux_div(model, u, ds, kappa=KAPPA):
    f0, _, f1, _ = _coeffs(model, u, kappa)
    lap = _lap(u, ds)
    out = torch.zeros_like(u)
    for d in (0, 1):
        k = u.shape[d] - 1
        L, R = (lambda a: a.narrow(d, 0, k)), (lambda a: a.narrow(d, 1, k))
        F = ((L(f0) + R(f0)) * (R(lap) - L(lap)) + (L(f1) + R(f1)) * (R(u) - L(u))) / (2.0 * ds)
        z = torch.zeros_like(u.narrow(d, 0, 1))
        F = torch.cat([z, F, z], d)
        out = out + (F.narrow(d, 1, k + 1) - F.narrow(d, 0, k + 1)) / ds
    return out


def _bands(model, u, ds, c, kappa=KAPPA):
    """Bands a..e of I + c J along dimension 0, shape (5, n, lines)."""
    f0, f0p, f1, f1p = _coeffs(model, u, kappa)
    lap = _lap(u, ds)
    L, R = (lambda a: a[:-1]), (lambda a: a[1:])
    Lam, Gam, Bf = (R(lap) - L(lap)) / ds, (R(u) - L(u)) / ds, 0.5 * (L(f1) + R(f1)) / ds
    z = torch.zeros_like(u[:1])
    kA = torch.cat([z, c / ds ** 4 * 0.5 * (L(f0) + R(f0)), z])
    P = torch.cat([z, c / ds * (0.5 * L(f0p) * Lam + 0.5 * L(f1p) * Gam - Bf), z])
    Q = torch.cat([z, c / ds * (0.5 * R(f0p) * Lam + 0.5 * R(f1p) * Gam + Bf), z])
    m, p = (lambda a: a[:-1]), (lambda a: a[1:])  # the faces below and above a cell
    a, e = m(kA).clone(), p(kA).clone()
    b = -p(kA) - 3.0 * m(kA) - m(P)
    d = -3.0 * p(kA) + p(Q) - m(kA)
    cc = 1.0 + 3.0 * p(kA) + p(P) + 3.0 * m(kA) - m(Q)
    cc[0] += b[0]
    d[0] += a[0]
    b[1] += a[1]
    cc[-1] += d[-1]
    b[-1] += e[-1]
    d[-2] += e[-2]
    a[:2], b[0], d[-1], e[-2:] = 0.0, 0.0, 0.0, 0.0
    return torch.stack([a, b, cc, d, e])


def _transposed(bands):
    a, b, c, d, e = bands
    z = torch.zeros_like(a[:2])
    return torch.stack([torch.cat([z, e[:-2]]), torch.cat([z[:1], d[:-1]]), c, torch.cat([b[1:], z[:1]]),
                        torch.cat([a[2:], z])])


def _solve(bands, rhs):
    """Gaussian elimination along dimension 0 of (5, n, lines) bands."""
    a, b, c, d, e = (x.numpy() for x in bands)
    x = rhs.numpy().copy()
    n = x.shape[0]
    al, be = np.empty_like(x), np.empty_like(x)
    zero = np.zeros_like(x[0])
    for p in range(n):
        al1, be1, x1 = (al[p - 1], be[p - 1], x[p - 1]) if p >= 1 else (zero, zero, zero)
        al2, be2, x2 = (al[p - 2], be[p - 2], x[p - 2]) if p >= 2 else (zero, zero, zero)
        gam = b[p] - a[p] * al2
        inv = 1.0 / (c[p] - a[p] * be2 - gam * al1)
        al[p] = (d[p] - gam * be1) * inv
        be[p] = e[p] * inv
        x[p] = (x[p] - a[p] * x2 - gam * x1) * inv
    for p in range(n - 2, -1, -1):
        x[p] -= al[p] * x[p + 1]
        if p + 2 < n:
            x[p] -= be[p] * x[p + 2]
    return torch.from_numpy(x)


def _cols(bands, rhs):
    return _solve(bands, rhs)


def _rows(bands, rhs):
    return _solve(bands, rhs.t().contiguous()).t().contiguous()


def _iteration(model, bn, uk, ds, dt, theta):
    """u_{k+1}, max|v/u_k|, max|G|."""
    c = theta * dt
    G = uk - bn + c * _flux_div(model, uk, ds)
    w = _cols(_bands(model, uk, ds, c), -G)
    v = _rows(_bands(model, uk.t().contiguous(), ds, c), w)
    return uk + v, float((v / uk).abs().max()), float(G.abs().max())


def _step(un, dt, theta=1.0, tol=1e-10, max_newton=5000):
    """One attempt of a step of the power-law film: (u^{n+1} or None, iterations)."""
    ds = MODELS["power"]["ds"]
    bn = un if theta == 1.0 else un - (1.0 - theta) * dt * _flux_div("power", un, ds)
    uk = un
    for _ in range(max_newton):
        uk, e, _ = _iteration("power", bn, uk, ds, dt, theta)
        if not bool((uk > 0.0).all()):
            return None
        if e < tol:
            return uk
    return None


def _exact_advance(case, seed):
    u = _film(_gen(seed), case["ny"], case["nx"], 1.0).cpu()
    dt, successes, masses, hmins = 0.1, 0, [], []
    for _ in range(case["steps"]):
        while True:
            new = _step(u, dt, max_newton=10 if case["adaptive"] else 5000)
            if new is not None:
                break
            successes = 0
            dt *= 0.5
        u = new
        successes += 1
        if case["adaptive"] and successes >= 5:
            dt, successes = min(1.1 * dt, 1.0), 0
        masses.append(math.fsum(u.numpy().ravel()))
        hmins.append(float(u.min()))
    out = {"h": u, "dt": dt}
    if case["mass"]:
        out.update(mass=masses, hmin=hmins)
    return out


def _exact_rollout(case, seed):
    base, p0, target = (t.cpu() for t in _rollout_inputs(case, seed))
    ds, dt, theta = MODELS["power"]["ds"], 0.1, case["theta"]
    c = theta * dt
    us = [base + p0]
    for _ in range(case["steps"]):
        us.append(_step(us[-1], dt, theta))
    lam = us[-1] - target
    loss = 0.5 * float(lam.square().sum())
    grad_k = 0.0

    def pull(u, mu):
        """(J_D(u)^T mu, mu . dD/dkappa(u))."""
        u = u.detach().requires_grad_()
        k = torch.tensor(KAPPA, dtype=torch.float64, requires_grad=True)
        return torch.autograd.grad((_flux_div("power", u, ds, k) * mu).sum(), (u, k))

    for n in range(case["steps"] - 1, -1, -1):
        u1, u0 = us[n + 1], us[n]
        by = _transposed(_bands("power", u1, ds, c))
        bx = _transposed(_bands("power", u1.t().contiguous(), ds, c))
        mu = lam.clone()
        for _ in range(200):
            z = _cols(by, _rows(bx, lam - mu - c * pull(u1, mu)[0]))
            mu = mu + z
            if float(z.abs().max()) <= 1e-10 * float(mu.abs().max()):
                break
        grad_k -= c * float(pull(u1, mu)[1])
        if theta < 1.0:
            j, k0 = pull(u0, mu)
            grad_k -= (1.0 - theta) * dt * float(k0)
            lam = mu - (1.0 - theta) * dt * j
        else:
            lam = mu
    return {"h": us[-1], "loss": torch.tensor(loss, dtype=torch.float64), "grad_p0": lam,
            "grad_kappa": torch.tensor(grad_k, dtype=torch.float64)}


def _exact_spectrum(case, seed):
    h, ds, h0, qmax = _spectrum_inputs(case, seed)
    n = case["n"]
    A = (torch.fft.fft2(h.cpu() - h0).abs() / n ** 2)
    w = torch.exp(-torch.arange(-4, 5, dtype=torch.float64) ** 2 / 2.0)
    w = w / w.sum()
    for d in (0, 1):
        A = sum(float(w[i]) * torch.roll(A, i - 4, d) for i in range(9))
    k = torch.fft.fftfreq(n, d=1.0 / n, dtype=torch.float64).round().to(torch.int64)
    m = (k[None, :] ** 2 + k[:, None] ** 2).reshape(-1).numpy()
    sums = np.bincount(m, weights=A.reshape(-1).numpy())
    counts = np.bincount(m)
    at = np.nonzero(counts)[0]
    q = 2.0 * math.pi * np.sqrt(at.astype(np.float64)) / (n * ds)
    keep = (at > 0) & (q <= qmax)
    return {"q": q[keep], "mean": sums[at[keep]] / counts[at[keep]], "count": counts[at[keep]].astype(np.int32)}


def exact(case, seed):
    path = case["path"]
    if path == "newton":
        m = MODELS[case["model"]]
        un, uk = (t.cpu() for t in _newton_inputs(case, seed))
        theta = case["theta"]
        bn = un if theta == 1.0 else un - (1.0 - theta) * m["dt"] * _flux_div(case["model"], un, m["ds"])
        u, e, r = _iteration(case["model"], bn, uk, m["ds"], m["dt"], theta)
        return {"u": u, "e": e, "r": r, "flags": None}
    if path == "advance":
        if case["nx"] * case["ny"] * case["steps"] > 3_000_000:
            return None  # minutes of CPU work
        return _exact_advance(case, seed)
    if path == "ensemble":
        return None  # the films' whole adaptive runs: minutes of CPU work
    if path == "rollout":
        return _exact_rollout(case, seed)
    if path == "penta":
        bands, rhs = (t.cpu() for t in _penta_inputs(case, seed))
        return _solve(_transposed(bands) if case["transposed"] else bands, rhs)
    return _exact_spectrum(case, seed)
