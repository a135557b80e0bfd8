"""Whole-line sweeps (one to several waves per line, cyclic reduction across the lanes) against the
oracle at the edges of their geometry: the shortest lines, one below / at / above a lane's 4, 8 and
16 positions, the lengths where the positions per lane and the waves per line change, the longest
columns and rows, and column counts that do not fill a workgroup."""
import numpy as np
import pytest
import torch

from paper_1806_10550_amd import synth
from paper_1806_10550_amd.lib import Ensemble, Grid

pytestmark = pytest.mark.gpu
DEV = "cuda:0"

# lengths on both sides of every change of geometry
EDGES = [4, 5, 7, 8, 9, 127, 128, 129, 255, 256, 257, 263, 384, 385, 511, 512, 513, 527, 640, 641, 768, 769,
         895, 897, 1023, 1024, 1025, 1039, 1280, 1281, 1536, 1537, 1792, 1793, 2047, 2048]


def one(orc, nx, ny, theta=1.0, model="power"):
    ds, dt, h0 = {"power": (0.67347, 0.2, 1.0), "nlc": (0.1325, 0.028, 0.5), "polymer": (0.126, 7.1e-4, 3.9),
                  "linear": (0.5, 0.05, 1.0)}[model]
    un = synth.noise_film(nx, ny, seed=nx + 3 * ny, h0=h0, amp=0.01 * h0)
    g = Grid(nx, ny, ds)
    if model == "power":
        g.set_model(10.0, 0.1, 3, 2)
        M = orc.Model(kappa=10.0, b=0.1, n=3.0, m=2.0)
    else:
        getattr(g, "set_model_" + model)()
        M = orc.Model.linear(1.0, 1.0) if model == "linear" else getattr(orc.Model, model)()
    g.set_scheme(theta=theta)
    if nx <= 8192:
        g.set_xsweep("row")
    u = torch.from_numpy(un).to(DEV)
    out = torch.empty_like(u)
    e, r, flags = g.newton_iteration(u, u, out, dt)
    ref, e_ref, r_ref = orc.adi_iteration(M, un, un, ds, dt, theta)
    got = out.cpu().numpy()
    # the parity tests' bound on one iterate: 1e-10 of the update (plus rounding of u itself)
    assert np.max(np.abs(got - ref)) <= 1e-10 * np.max(np.abs(ref - un)) + 4e-16 * h0
    assert flags == 0
    assert e == pytest.approx(e_ref, rel=1e-8)
    assert r == pytest.approx(r_ref, rel=1e-8)
    g.close()


@pytest.mark.parametrize("n", EDGES)
def test_columns_match_oracle(orc, n):
    one(orc, 6, n)


@pytest.mark.parametrize("n", EDGES + [2304, 2305, 2688, 2689, 3072, 3073, 3584, 3585, 4096, 5000, 8191, 8192])
def test_rows_match_oracle(orc, n):
    one(orc, n, 5)


@pytest.mark.parametrize("model,theta", [("nlc", 0.5), ("polymer", 1.0), ("linear", 0.5)])
@pytest.mark.parametrize("nx,ny", [(67, 130), (300, 517), (1030, 300), (21, 1500)])
def test_models_match_oracle(orc, model, theta, nx, ny):
    one(orc, nx, ny, theta, model)


@pytest.mark.parametrize("ny", [1025, 1280, 1281, 1536, 1537, 1792, 1793, 2048, 2049])
def test_nlc_long_columns_match_oracle(orc, ny):
    one(orc, 9, ny, 0.5, "nlc")


@pytest.mark.parametrize("transposed", [False, True])
@pytest.mark.parametrize("n", EDGES + [2049, 3072, 3073, 4095, 4096])
def test_stored_band_lines_match_oracle(orc, n, transposed):
    """The whole-line stored-band solver with one line, one short of and one past a workgroup's lines
    (diagonally dominant bands; the bound of the solver tests)."""
    from paper_1806_10550_amd.lib import penta_solve
    rng = np.random.default_rng(n)
    for nl in (1, 3, 5):
        bands = rng.standard_normal((5, n, nl))
        bands[2] = 6.0 + rng.random((n, nl))
        bands[0, :2] = bands[1, :1] = bands[3, n - 1:] = bands[4, n - 2:] = 0.0
        rhs = rng.standard_normal((n, nl))
        b, r = torch.from_numpy(bands).to(DEV), torch.from_numpy(rhs).to(DEV)
        x = penta_solve(b, r, torch.empty_like(r), transposed=transposed, variant="line").cpu().numpy()
        for l in range(nl):
            band = np.ascontiguousarray(bands[:, :, l])
            ref = orc.band_solve(orc.band_transpose(band) if transposed else band, rhs[:, l].copy())
            assert np.max(np.abs(x[:, l] - ref)) <= 1e-12 * max(1.0, np.max(np.abs(ref))), (n, nl, l)


@pytest.mark.parametrize("dt", [1e-9, 1e-3, 10.0])
@pytest.mark.parametrize("nx,ny,xsweep", [(100, 90, "row"), (512, 300, "row"), (1500, 700, "row"), (640, 1300, "row"),
                                          (4200, 70, "row"), (200, 2600, "partitioned")])
def test_weak_and_strong_coupling_match_oracle(orc, nx, ny, xsweep, dt):
    """The reduction takes no step or many. Bound: pivots good to 11 units of 2^-53 and the norms of the
    two factors, 1 + 16 c / ds^4 max f0 each (at least the suite's 1e-12). It holds while I + c J is
    definite; at dt = 1e3 the film's growing modes make it indefinite, and neither these solvers nor a
    merge tree or the partition meet it (1e-7 to 1e-3 of the update)."""
    ds = 0.67347
    un = synth.noise_film(nx, ny, seed=nx + ny, amp=0.01)
    g = Grid(nx, ny, ds)
    g.set_model(10.0, 0.1, 3, 2)
    g.set_xsweep(xsweep)
    u = torch.from_numpy(un).to(DEV)
    out = torch.empty_like(u)
    g.newton_iteration(u, u, out, dt)
    uo = orc.adi_iteration(orc.Model(kappa=10.0, b=0.1, n=3.0, m=2.0), un, un, ds, dt, 1.0)[0]
    c = dt * 1.05 / ds ** 4
    tol = max(1e-12, 11 * 2.0 ** -53 * 2 * (1.0 + 16.0 * c))
    assert np.max(np.abs(out.cpu().numpy() - uo)) <= tol * np.max(np.abs(uo))
    g.close()


@pytest.mark.parametrize("bad", [float("nan"), float("inf")])
@pytest.mark.parametrize("xsweep", ["row", "partitioned"])
@pytest.mark.parametrize("nx,ny", [(100, 90), (512, 300), (1500, 700), (600, 1500), (70, 2600), (4200, 70)])
def test_non_finite_right_side_reaches_the_whole_film(nx, ny, xsweep, bad):
    """u^n non-finite in one cell, u_k finite (so are all bands): the elimination carries it through that
    column and then through every row, however weakly the cells are coupled."""
    un = synth.noise_film(nx, ny, seed=nx + ny, amp=0.01)
    g = Grid(nx, ny, 0.67347)
    g.set_model(10.0, 0.1, 3, 2)
    g.set_xsweep(xsweep)
    uk = torch.from_numpy(un).to(DEV)
    u = uk.clone()
    u[ny // 3, nx // 2] = bad
    out = torch.zeros_like(uk)
    _, _, flags = g.newton_iteration(u, uk, out, 0.2)
    assert flags != 0
    assert not bool(torch.isfinite(out).any())
    g.close()


@pytest.mark.parametrize("transposed", [False, True])
@pytest.mark.parametrize("n", [64, 248, 256, 500, 777, 1500])
def test_stored_band_lines_are_as_exact_as_elimination(n, transposed):
    """Bands like those of a film's I + c J: the error of a plain elimination in 64 bits is 2.2e-16 of the
    solution's 2-norm (mean over many lines); the bound leaves a quarter of 2^-53 to the reduction, less
    than its steps' errors (3.1e-16 with four cells a lane) unless the pairs' equations remove them."""
    from paper_1806_10550_amd.lib import penta_solve
    rng = np.random.default_rng(n)
    nl = 64
    k = 0.5 * (1.0 + 0.5 * rng.uniform(-1.0, 1.0, (n, nl)))
    e = 0.05 * rng.uniform(-1.0, 1.0, (2, n, nl))
    bands = np.stack([k, -4.0 * k + e[0], 1.0 + 6.0 * k, -4.0 * k + e[1], k])
    bands[0, :2] = bands[1, :1] = bands[3, n - 1:] = bands[4, n - 2:] = 0.0
    rhs = rng.uniform(-1.0, 1.0, (n, nl))
    b, r = torch.from_numpy(bands).to(DEV), torch.from_numpy(rhs).to(DEV)
    x = penta_solve(b, r, torch.empty_like(r), transposed=transposed, variant="line").cpu().numpy()
    # exact solution by elimination in extended precision
    m = bands.astype(np.longdouble)
    if transposed:
        t = np.zeros_like(m)
        for d in range(5):
            o = d - 2 # row q's entry at column q + o is the plain matrix's (q + o, q)
            lo, hi = max(0, -o), n - max(0, o)
            t[d, lo:hi] = m[4 - d, lo + o:hi + o]
        m = t
    al, be, z = (np.zeros((n + 2, nl), np.longdouble) for _ in range(3)) # rows shifted by two
    for q in range(n):
        g = m[1, q] - m[0, q] * al[q]
        mu = m[2, q] - m[0, q] * be[q] - g * al[q + 1]
        al[q + 2] = (m[3, q] - g * be[q + 1]) / mu
        be[q + 2] = m[4, q] / mu
        z[q + 2] = (rhs[q] - m[0, q] * z[q] - g * z[q + 1]) / mu
    ref = np.zeros((n + 2, nl), np.longdouble)
    for q in range(n - 1, -1, -1):
        ref[q] = z[q + 2] - al[q + 2] * ref[q + 1] - be[q + 2] * ref[q + 2]
    ref = ref[:n]
    err = float(np.sqrt(np.sum((x - ref) ** 2) / np.sum(ref ** 2)))
    assert err <= 2.2e-16 + 0.25 * 2.0 ** -53, err


@pytest.mark.parametrize("nx,ny", [(4097, 129), (4200, 70), (9, 2049), (66, 4160), (5, 4161), (3, 8256), (3, 8257),
                                   (130, 2304)])
def test_partitioned_chains_match_oracle(orc, nx, ny):
    """Interface systems on both sides of the rules between cyclic reduction (one and two waves per line)
    and the serial chain: 2, 64, 65, 66, 129 and 130 segments, 4096 and more lines."""
    ds, dt = 0.67347, 0.2
    nx = max(nx, 4)
    un = synth.noise_film(nx, ny, seed=nx + ny, amp=0.01)
    g = Grid(nx, ny, ds)
    g.set_model(10.0, 0.1, 3, 2)
    g.set_xsweep("partitioned")
    u = torch.from_numpy(un).to(DEV)
    out = torch.empty_like(u)
    e, r, flags = g.newton_iteration(u, u, out, dt)
    ref, e_ref, _ = orc.adi_iteration(orc.Model(kappa=10.0, b=0.1, n=3.0, m=2.0), un, un, ds, dt, 1.0)
    assert np.max(np.abs(out.cpu().numpy() - ref)) <= 1e-10 * np.max(np.abs(ref - un)) + 4e-16
    assert flags == 0 and e == pytest.approx(e_ref, rel=1e-8)
    g.close()


def test_ensemble_of_every_line_class_equals_single_films():
    """One film per geometry class of the columns and rows (and one that takes tiles), bit for bit."""
    shapes = [(100, 90), (300, 60), (500, 300), (600, 500), (700, 600), (800, 700), (1000, 800), (1200, 900), (30, 1200),
              (1500, 40), (40, 1500), (1700, 20), (20, 1700), (2000, 10), (10, 2000), (2200, 8), (2500, 40), (3000, 9),
              (3500, 8), (4000, 24), (9, 2100)]
    nx, ny = [a for a, _ in shapes], [b for _, b in shapes]
    ds = [0.67347] * len(shapes)
    kap = [10.0 + i for i in range(len(shapes))]
    ens = Ensemble(nx, ny, ds, kap)
    ens.set_scheme(theta=0.5, tol=1e-10)
    h0 = [synth.noise_film(a, b, seed=i, amp=0.01) for i, (a, b) in enumerate(shapes)]
    packed = torch.empty(ens.size, dtype=torch.float64, device=DEV)
    for f, h in enumerate(h0):
        ens.view(packed, f).copy_(torch.from_numpy(h))
    ens.bind(packed)
    st, _, sts, its = ens.step(2, 0.1)
    assert st == 0 and not any(sts)
    for f in range(len(shapes)):
        g = Grid(nx[f], ny[f], ds[f])
        g.set_model(kap[f], 0.1, 3, 2)
        g.set_scheme(theta=0.5, tol=1e-10)
        g.set_xsweep(ens.xsweep(f))
        h = torch.from_numpy(h0[f]).to(DEV)
        g.bind(h)
        _, log = g.advance(2, 0.1, log=True)
        assert torch.equal(ens.view(packed, f), h), shapes[f]
        assert its[f] == sum(x["total_iters"] for x in log)
        g.close()
