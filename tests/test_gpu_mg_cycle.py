"""One multigrid cycle against its definition: the restriction and the
interpolation as dense numpy rows, the coarsest grid's damped sweeps as the
PT iterations of a grid of its own.  Coarsest grids that one block holds
(smallest, ragged, largest by cells and by LDS) and ones that take the
ordinary sweeps; coarse grids of one and of several planes per chunk."""
import dataclasses

import numpy as np
import pytest

from paper_2207_08716_amd import inputs, schedules
from paper_2207_08716_amd.grid import Grid

pytestmark = pytest.mark.gpu

STATE = ("vx", "vy", "vz", "pt", "pf")
FACE = {"vx": 2, "vy": 1, "vz": 0}                       # the array axis a velocity is normal to


def _p(nf, nc, face):
    """Interpolation from nc coarse to nf fine points of an axis, (fine, coarse)."""
    i = np.arange(nf + face)
    u = i * nc / nf if face else np.clip((i + 0.5) * nc / nf - 0.5, 0, nc - 1)
    j = np.minimum(np.floor(u).astype(int), nc - 1 if face else max(nc - 2, 0))
    m = np.zeros((nf + face, nc + face))
    m[i, j] += 1 - (u - j)
    m[i, j + 1] += u - j
    return m


def _r(nf, nc, face):
    """Restriction: the transpose with rows of sum 1, no walls' faces."""
    m = _p(nf, nc, face).T.copy()
    if face:
        m[:, [0, -1]] = 0
        m[[0, -1]] = 0
    s = m.sum(1, keepdims=True)
    return np.divide(m, s, out=np.zeros_like(m), where=s > 0)


def _apply(rows, v):
    return np.einsum("ak,bj,ci,kji->abc", *rows, v, optimize=True)


def _mean(rows, v, kind):
    if kind == 0:
        return _apply(rows, v)
    return 1 / _apply(rows, 1 / v) if kind == 1 else np.exp(_apply(rows, np.log(v)))


@pytest.mark.parametrize("shape,eta_mean", [
    ((4, 4, 4), 0), ((5, 4, 7), 1), ((16, 16, 16), 2), ((17, 5, 9), 0), ((20, 19, 20), 1), ((8, 8, 100), 0),
    ((8, 8, 110), 2), ((40, 8, 40), 0), ((30, 27, 25), 1), ((100, 90, 60), 0)])
def test_a_cycle_matches_its_definition(shape, eta_mean):
    nx, ny, nz = shape
    cfg = dataclasses.replace(inputs.config_mixed(nx), nx=nx, ny=ny, nz=nz)
    g = schedules.make_grid(cfg, inputs.initial_fields(cfg))
    g.begin_step(False)
    g.refresh(1.0, 1.0)
    for _ in range(20):
        g.iteration(False)
    x0 = {n: g.get(n) for n in STATE}
    sweeps = 50
    g.solve_mg(1e-300, 0, levels=2, nu1=1, nu2=1, coarse_sweeps=sweeps, krylov=0, eta_mean=eta_mean)
    x1 = {n: g.get(n) for n in STATE}
    g.residual()
    res = dict(zip(STATE, g.residual_fields()))
    coef = {n: g.get(n) for n in ("kc", "eta", "mus", "lp")}
    (_, coarse) = g.mg_levels()

    def rows(make, face=None):
        return [make(f, c, a == face) for a, (f, c) in enumerate(zip(shape[::-1], coarse[::-1]))]

    ph = cfg.phys.replace(rhofg=0.0, rhosg=0.0)
    h = Grid(ph, *coarse)
    h.load_initial(np.full(coarse[::-1], ph.phi0))
    h.begin_step(False)
    h.refresh(1.0, 1.0)
    for n, kind in (("kc", 1), ("eta", eta_mean), ("mus", 0), ("lp", 0)):
        h.set(n, _mean(rows(_r), coef[n].astype(np.float64), kind))
    for n in STATE:
        h.set(n, 0.0)
    for n, fo in (("vx", "fox"), ("vy", "foy"), ("vz", "foz")):
        h.set(fo, _apply(rows(_r, FACE[n]), res[n].astype(np.float64)))
    # beta_d/dt (alpha pfo - pto) = r_Pt, beta_d/dt (alpha pto - alpha/B pfo) = r_Pf
    k = ph.beta_d / ph.dt
    a, b = (_apply(rows(_r), res[n].astype(np.float64)) for n in ("pt", "pf"))
    inv = np.linalg.inv(k * np.array([[-1, ph.alpha], [ph.alpha, -ph.alpha / ph.B]]))
    h.set("pto", inv[0, 0] * a + inv[0, 1] * b)
    h.set("pfo", inv[1, 0] * a + inv[1, 1] * b)
    for _ in range(sweeps):
        h.iteration(False)
    want = {}
    for n in STATE:
        e = _apply(rows(_p, FACE.get(n)), h.get(n))
        if n in FACE:
            np.moveaxis(e, FACE[n], 0)[[0, -1]] = 0
        want[n] = x1[n] + e
    for n in STATE:
        g.set(n, want[n])
    g.solve_mg(1e-300, 0, levels=2, nu1=2, nu2=0, coarse_sweeps=sweeps, krylov=0, eta_mean=eta_mean)
    want = {n: g.get(n) for n in STATE}
    for n in STATE:
        g.set(n, x0[n])
    g.solve_mg(1e-300, 1, levels=2, nu1=1, nu2=1, coarse_sweeps=sweeps, krylov=0, eta_mean=eta_mean)
    # some hundred roundings of 1.1e-16 per sweep and value over 50 sweeps, on
    # the correction's and the state's scale
    for n in STATE:
        d = np.abs(g.get(n) - want[n]).max()
        s = max(np.abs(want[n]).max(), np.abs(want[n] - x1[n]).max())
        print(shape, n, d / s, flush=True)
        assert np.abs(want[n] - x1[n]).max() > 1e-6 * s
        assert d <= 1e-11 * s, n
