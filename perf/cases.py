"""The workloads by which this framework's speed is judged: what its users run, through its public entry points.

Sizes, parameters and input recipes are those of ``inputs.py``, the tests and ``bench.py`` (the 32^3 parity workload,
the 511^3 two-anomaly workload, the sheared production box, the reactive porosity waves with their 506 x 506 x 2042
grid, the adjoint workload), with odd and ragged grids among them.  Inputs are made on the GPU from the seed.

``exact`` repeats a case's arithmetic in plain torch, in 64 bits, for the cases with a fixed or small number of
iterations: none of the library's kernels takes part in it.
"""
import math

import torch

from paper_2207_08716_amd import autograd, inputs
from paper_2207_08716_amd.grid import Grid
from paper_2207_08716_amd.waves import Waves

DEV = "cuda"


def listed():
    return [
        # the parity workload of the tests and of the paper's small runs: one refresh cycle (a refresh, then 15
        # iterations, the last with norms) on the smallest grid in use, where launches and latency count
        {"name": "thesis_32", "kind": "thesis", "load": "parity", "nx": 32, "ny": 32, "nz": 32, "iters": 15},
        # the same schedule on an ordinary ragged grid with a permeability field and the yield cap
        {"name": "thesis_173x131x97", "kind": "thesis", "load": "mixed", "nx": 173, "ny": 131, "nz": 97, "iters": 30},
        # the benchmark's step: one refresh cycle at 511^3
        {"name": "thesis_511", "kind": "thesis", "load": "mixed", "nx": 511, "ny": 511, "nz": 511, "iters": 15},
        # a physical step of the production set-up: begin_step with the stress-history rule, power law, shear
        {"name": "production_255x255x510", "kind": "production", "nx": 255, "ny": 255, "nz": 510, "iters": 15},
        # a Picard step of one stage by FP64 sweeps to a relative residual, as the small tests and inversions run it
        {"name": "linear_40", "kind": "picard", "solver": "fp64", "load": "picard", "nx": 40, "ny": 40, "nz": 40,
         "stages": 1, "rtol": 1e-8},
        # the same by FP32 sweeps inside FP64 defect correction, at a size where the mixed solver is the usual choice
        {"name": "mixed_95", "kind": "picard", "solver": "mixed", "load": "mixed", "nx": 95, "ny": 95, "nz": 95,
         "stages": 1, "rtol": 1e-10},
        # a whole physical step (5 Picard stages to 1e-8) by multigrid: the benchmark's time to tolerance
        {"name": "mg_127", "kind": "picard", "solver": "mg", "load": "mixed", "nx": 127, "ny": 127, "nz": 127,
         "stages": 5, "rtol": 1e-8},
        # one multigrid stage on a large grid that does not halve evenly
        {"name": "mg_300x255x201", "kind": "picard", "solver": "mg", "load": "mixed", "nx": 300, "ny": 255, "nz": 201,
         "stages": 1, "rtol": 1e-8},
        # the production box by Krylov-accelerated cycles (8 stored directions), one stage
        {"name": "mgk_production_95x95x190", "kind": "picard", "solver": "mgk", "load": "production", "nx": 95,
         "ny": 95, "nz": 190, "stages": 1, "rtol": 1e-8},
        # reactive porosity waves: a small box, and the paper's full grid
        {"name": "reactive_31x31x124", "kind": "reactive", "nx": 31, "ny": 31, "nz": 124, "da": 100.0, "iters": 20},
        {"name": "reactive_506x506x2042", "kind": "reactive", "nx": 506, "ny": 506, "nz": 2042, "da": 100.0,
         "iters": 10},
        # one inversion step: a stage solve, the sensor misfit and its gradient with respect to ln k0 (forward and
        # backward through torch.autograd)
        {"name": "adjoint_31", "kind": "adjoint", "nx": 31, "ny": 31, "nz": 31, "sensors": 16, "rtol": 1e-10},
    ]


def _size(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["thesis", "thesis", "production", "fp64", "mixed", "mg", "mg", "mgk", "reactive", "reactive",
                       "adjoint"])
    if kind == "thesis":
        n = _size(rng, 16, 420)
        dims = [max(12, min(511, int(n * rng.uniform(0.6, 1.4)))) for _ in range(3)]
        return {"kind": "thesis", "load": rng.choice(["parity", "mixed", "picard"]), "nx": dims[0], "ny": dims[1],
                "nz": dims[2], "iters": 15 * rng.randint(1, 2)}
    if kind == "production":
        n = _size(rng, 16, 255)
        return {"kind": "production", "nx": n, "ny": max(12, n - rng.randint(0, 9)), "nz": 2 * n - rng.randint(0, 3),
                "iters": 15}
    if kind in ("fp64", "mixed"):
        n = _size(rng, 14, 44) if kind == "fp64" else _size(rng, 20, 90)
        return {"kind": "picard", "solver": kind, "load": rng.choice(["picard", "mixed"]), "nx": n,
                "ny": max(12, n - rng.randint(0, 5)), "nz": max(12, n - rng.randint(0, 5)), "stages": 1,
                "rtol": 1e-8 if kind == "fp64" else 1e-10}
    if kind == "mg":
        n = _size(rng, 20, 290)
        dims = [max(18, int(n * rng.uniform(0.75, 1.0))) for _ in range(3)]
        return {"kind": "picard", "solver": "mg", "load": rng.choice(["picard", "mixed"]), "nx": dims[0],
                "ny": dims[1], "nz": dims[2], "stages": rng.randint(1, 2), "rtol": 1e-8}
    if kind == "mgk":
        n = _size(rng, 18, 90)
        return {"kind": "picard", "solver": "mgk", "load": "production", "nx": n, "ny": n, "nz": 2 * n - rng.randint(0, 1),
                "stages": 1, "rtol": 1e-8}
    if kind == "reactive":
        n = _size(rng, 12, 380)
        return {"kind": "reactive", "nx": n, "ny": max(10, n - rng.randint(0, 7)), "nz": 4 * n - rng.randint(0, 5),
                "da": rng.choice([100.0, 0.01]), "iters": 10 * rng.randint(1, 2)}
    n = _size(rng, 10, 31)
    return {"kind": "adjoint", "nx": n, "ny": n, "nz": max(10, n - rng.randint(0, 3)), "sensors": rng.randint(4, 32),
            "rtol": 1e-10}


# ---- inputs -----------------------------------------------------------------

def _phys(case):
    kind = case["kind"]
    if kind == "reactive":
        return inputs.config_reactive(8, da=case["da"]).phys
    if kind == "adjoint":
        return inputs.config_adjoint(8).phys
    load = "production" if kind == "production" else case["load"]
    return {"parity": inputs.config_parity, "picard": inputs.config_fp64_picard, "mixed": inputs.config_mixed,
            "production": lambda n: inputs.config_production(n, n, 2 * n)}[load](8).phys


def _inputs(case, seed):
    """(porosity, ln k0 or None) on the GPU: the recipes of inputs.py with the anomalies, the noise and the
    permeability drawn from the seed."""
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed))
    ph = _phys(case)
    shape = (case["nz"], case["ny"], case["nx"])
    u = torch.rand(16, generator=g, device=DEV, dtype=torch.float64).tolist()
    kind, load = case["kind"], case.get("load")
    if kind == "reactive":
        anomalies = [((6.25 + u[0] - 0.5, 6.25 + u[1] - 0.5, 5.0 + u[2]), 1.5, (1.5,) * 3),
                     ((6.25 + u[3] - 0.5, 6.25 + u[4] - 0.5, 11.5 + u[5]), 0.75, (1.5,) * 3)]
    elif kind == "production" or load == "production":
        anomalies = [((14.0 + 2 * u[0], 14.0 + 2 * u[1], 11.0 + 2 * u[2]), 1.0, (7.0, 7.0, 1.75))]
    elif load == "mixed":
        anomalies = [((0.3 + 0.4 * u[0], 0.3 + 0.4 * u[1], 0.15 + 0.3 * u[2]), 2.0, (0.1,) * 3),
                     ((0.3 + 0.4 * u[3], 0.3 + 0.4 * u[4], 0.15 + 0.3 * u[5]), 1.5, (0.1,) * 3)]
    else:
        anomalies = [((0.4 + 0.2 * u[0], 0.4 + 0.2 * u[1], 0.2 + 0.1 * u[2]), 2.0, (0.1,) * 3)]
    phi = torch.full(shape, ph.phi0, dtype=torch.float64, device=DEV)
    for centre, amp, width in anomalies:
        # separable Gaussian: exp of a sum, built axis by axis
        e = [torch.exp(-(((torch.arange(n, dtype=torch.float64, device=DEV) + 0.5) * (length / n) - c) / w) ** 2)
             for n, length, c, w in zip(shape[::-1], (ph.lx, ph.ly, ph.lz), centre, width)]
        phi += (amp * ph.phi0 * e[2])[:, None, None] * e[1][None, :, None] * e[0][None, None, :]
    if kind != "reactive" and kind != "production" and load != "production":
        phi *= 1.0 + 1e-3 * (2.0 * torch.rand(shape, generator=g, device=DEV, dtype=torch.float64) - 1.0)
    logk = None
    if load in ("mixed", "picard") or kind == "adjoint":
        logk = math.log(ph.kmuf0) + 0.5 * torch.randn(shape, generator=g, device=DEV, dtype=torch.float64)
    if kind == "adjoint":
        for d in range(3):          # a correlated field: running means of the white noise, back to sigma 0.5
            k = max(1, shape[d] // 8) * 2 + 1
            x = logk.movedim(d, -1)
            x = torch.nn.functional.pad(x.reshape(1, -1, x.shape[-1]), (k // 2, k // 2), mode="replicate")
            x = torch.nn.functional.avg_pool1d(x, k, 1)
            logk = x.reshape(logk.movedim(d, -1).shape).movedim(-1, d).contiguous()
        logk = 0.5 * logk / logk.std()
    return phi, logk


def prepare(case, seed):
    phi, logk = _inputs(case, seed)
    ph = _phys(case)
    nx, ny, nz = case["nx"], case["ny"], case["nz"]
    if case["kind"] == "reactive":
        w = Waves(ph, nx, ny, nz, phi.cpu().numpy())
        w.begin_step()
        return {"case": case, "waves": w}
    g = Grid(ph, nx, ny, nz, k0field=logk is not None)
    if logk is not None:
        g.set_log_k0(logk)
    g.reset_state(phi)
    state = {"case": case, "grid": g, "phi": phi}
    if case["kind"] == "thesis":
        g.begin_step(False)
    elif case["kind"] == "production":
        for _ in range(2):          # the history of the first steps: the pass is an ordinary later step
            g.begin_step(True)
            g.iterate(case["iters"])
    elif case["kind"] == "picard":
        if case["solver"] == "mixed":
            g.enable_mixed()
        elif case["solver"] in ("mg", "mgk"):
            g.enable_mg(krylov=8 if case["solver"] == "mgk" else 0)
    else:
        sensors = inputs.sensor_cells(int(seed) % 1000, case["sensors"], (nz, ny, nx))
        d_obs = [0.01 * (s % 7) for s in range(case["sensors"])]
        g.enable_adjoint(max(64, case["sensors"]))
        state["problem"] = autograd.StageProblem(g, phi, sensors, d_obs, rtol=case["rtol"])
        state["logk"] = logk.requires_grad_(True)
    return state


FIELDS = ("vx", "vy", "vz", "pt", "pf", "lp")


def run(state):
    case = state["case"]
    if case["kind"] == "reactive":
        w = state["waves"]
        w.iterate(case["iters"])
        return {name: w.view(name) for name in ("xs", "pf", "phi", "dpfdt")}
    g = state["grid"]
    if case["kind"] == "adjoint":
        J = autograd.LogKMisfit.apply(state["logk"], state["problem"])
        (grad,) = torch.autograd.grad(J, state["logk"])
        return {"J": J.detach(), "grad": grad}
    if case["kind"] == "thesis":
        g.iterate(case["iters"])
        return {name: g.view(name) for name in FIELDS + ("eta", "mn")}
    if case["kind"] == "production":
        g.begin_step(True)
        g.iterate(case["iters"])
        return {name: g.view(name) for name in FIELDS + ("eta", "mn")}
    # a step of the Picard schedule from the initial state (a converged state would end it at once)
    g.reset_state(state["phi"])
    solver = "mg" if case["solver"] == "mgk" else case["solver"]
    _sweeps, rho, ok = g.picard_step(False, case["stages"], case["rtol"], solver=solver,
                                     max_iter=500 if solver == "mg" else 2_000_000)
    if not ok:
        raise RuntimeError("the Picard step did not converge: rho %.3e" % rho)
    return {name: g.view(name) for name in FIELDS}


# ---- the work a pass cannot do without ------------------------------------------

# Values moved per cell by one iteration: the two-phase iteration reads three velocities and their previous iterate,
# two pressures and their old values, the porosity and its old value, three history divergences and three
# coefficients, and writes the six iterated fields; a linear iteration keeps the porosity (5 written, its old value
# not read).  About 300 operations per cell.
THESIS, LINEAR, FLOP = 18 + 6, 17 + 5, 300.0
# A refresh: three velocities, viscosity, six history components, both pressures, porosity, k0 and the two relaxed
# coefficients in; k, eta_phi, Mn, mu_s and three history divergences out.
REFRESH = 16 + 7


def work(case):
    cells = float(case["nx"] * case["ny"] * case["nz"])
    kind = case["kind"]
    if kind == "reactive":      # four fields read and written, three old-step fields read
        return {"bytes": 88.0 * cells * case["iters"], "flops": 90.0 * cells * case["iters"]}
    if kind in ("thesis", "production"):
        refreshes = (case["iters"] + 14) // 15
        extra = 20.0 if kind == "production" else 0.0      # old values, stress history
        return {"bytes": 8.0 * cells * (THESIS * case["iters"] + REFRESH * refreshes + extra),
                "flops": FLOP * cells * case["iters"]}
    # solves to a tolerance: iterations as the method needs them (they grow with the cells per axis)
    n = max(case["nx"], case["ny"], case["nz"])
    if kind == "adjoint":
        sweeps = 2 * 160.0 * n
        return {"bytes": 8.0 * cells * LINEAR * sweeps, "flops": FLOP * cells * sweeps}
    if case["solver"] in ("fp64", "mixed"):
        sweeps, size = (110.0 * n, 8.0) if case["solver"] == "fp64" else (280.0 * n, 4.0)
        return {"bytes": size * cells * LINEAR * sweeps, "flops": FLOP * cells * sweeps}
    # a V-cycle: nine sweeps' worth per grid, the coarser grids 1/7 of the finest
    cycles = (24.0 if case["stages"] == 1 else 13.0 * case["stages"])
    per = 9 * LINEAR * 8.0 * 8.0 / 7.0
    return {"bytes": cells * per * cycles, "flops": 9 * FLOP * cells * cycles * 8.0 / 7.0}


# ---- the same arithmetic in plain torch, in 64 bits --------------------------------

def exact(case, seed):
    if case["kind"] == "reactive":
        phi, _ = _inputs(case, seed)
        return _exact_reactive(_phys(case), phi, case["iters"])
    if case["kind"] in ("thesis", "production"):
        phi, logk = _inputs(case, seed)
        s = _TwoPhase(_phys(case), phi, logk)
        for _ in range(3 if case["kind"] == "production" else 1):
            s.begin_step(case["kind"] == "production")
            s.iterate(case["iters"])
        return {name: getattr(s, name) for name in FIELDS + ("eta", "mn")}
    if case["kind"] == "picard" and case["solver"] == "fp64" and max(case["nx"], case["ny"], case["nz"]) <= 44:
        phi, logk = _inputs(case, seed)
        s = _TwoPhase(_phys(case), phi, logk)
        s.begin_step(False)
        for _ in range(case["stages"]):
            s.refresh(1.0, 1.0)
            s.solve(case["rtol"])
            s.porosity_step()
        return {name: getattr(s, name) for name in FIELDS}
    return None      # thousands of iterations, cycles or a gradient: too long in plain torch


def _exact_reactive(p, phi, iters):
    nz, ny, nx = phi.shape
    d = (p.lz / nz, p.ly / ny, p.lx / nx)
    h = min(d)
    xs = torch.full_like(phi, 0.5 * p.xs_max)
    pf = torch.zeros_like(phi)
    dp = torch.zeros_like(phi)
    xso, pfo, phio = xs, pf, phi
    rho_term = 1.0 - p.rho_s / (p.rho_f * (1.0 + p.delta_x))
    dtau = 0.0
    for it in range(iters):
        k = p.k_muf0 * (phi / p.phi0) ** 3
        bp = phi * p.beta_f + p.beta_d - (1.0 + phi) * p.beta_s
        if it % p.nup == 0:
            dtau = h * h / p.c_pf / float((k / bp).max())
        divq = torch.zeros_like(phi)
        for axis in range(3):
            n = phi.shape[axis]
            lo, hi = [t.narrow(axis, 0, n - 1) for t in (k, pf)], [t.narrow(axis, 1, n - 1) for t in (k, pf)]
            q = (hi[1] - lo[1]) / d[axis]
            if axis == 0:
                q -= p.rho_f * p.g
            q *= -0.5 * (lo[0] + hi[0])
            divq.narrow(axis, 0, n - 1).add_(q, alpha=1.0 / d[axis])
            divq.narrow(axis, 1, n - 1).sub_(q, alpha=1.0 / d[axis])
            del lo, hi, q
        del k
        dxs = (torch.clamp(p.beta_x * pf + 0.5 * p.xs_max, 0.0, p.xs_max) - xs) / p.tau
        comp = -pf / (p.eta * (1.0 - phi))
        rate = (1.0 + p.delta_x) / (1.0 - xs) * dxs
        phin = torch.clamp(phio + p.dt * (1.0 - phi) * ((p.beta_d - p.beta_s / (1.0 - phi)) * dp - comp - rate),
                           p.phi_min, p.phi_max)
        dpn = (-divq + comp + rho_term * (1.0 - phi) * rate) / bp
        del divq, comp, rate, bp
        pf = pf + dtau * dp - dtau * (pf - pfo) / p.dt
        xs = xso + p.dt * dxs
        phi, dp = phin, dpn
        del dxs, phin, dpn
    return {"xs": xs, "pf": pf, "phi": phi, "dpfdt": dp}


def _dif(t, axis):
    """Differences along an axis (0: z, 1: y, 2: x) between neighbours: one fewer."""
    n = t.shape[axis]
    return t.narrow(axis, 1, n - 1) - t.narrow(axis, 0, n - 1)


def _avg(t, axis):
    n = t.shape[axis]
    return 0.5 * (t.narrow(axis, 1, n - 1) + t.narrow(axis, 0, n - 1))


def _inner(t, axis):
    """Without the first and last entry along an axis."""
    return t.narrow(axis, 1, t.shape[axis] - 2)


def _wall(t, axis):
    """A zero entry before and after, along an axis."""
    pad = [0] * 6
    pad[2 * (2 - axis)] = pad[2 * (2 - axis) + 1] = 1
    return torch.nn.functional.pad(t, pad)


class _TwoPhase:
    """The two-phase pseudo-transient iteration on compact (z, y, x) arrays: thesis schedule, linear stage solve."""

    def __init__(self, ph, phi, logk):
        self.p = ph
        nz, ny, nx = phi.shape
        self.n = (nz, ny, nx)
        self.d = (ph.lz / nz, ph.ly / ny, ph.lx / nx)
        new = lambda *s: torch.zeros(s, dtype=torch.float64, device=phi.device)  # noqa: E731
        self.vz, self.vy, self.vx = new(nz + 1, ny, nx), new(nz, ny + 1, nx), new(nz, ny, nx + 1)
        self.rz, self.ry, self.rx = new(nz - 1, ny, nx), new(nz, ny - 1, nx), new(nz, ny, nx - 1)
        self.pt, self.pf = new(nz, ny, nx), new(nz, ny, nx)
        self.pto, self.pfo = self.pt, self.pf
        self.lp = torch.log(1.0 - phi)
        self.lpo = self.lp
        self.so = [new(nz, ny, nx) for _ in range(3)]                       # zz, yy, xx
        self.syz, self.sxz, self.sxy = new(nz + 1, ny + 1, nx), new(nz + 1, ny, nx + 1), new(nz, ny + 1, nx + 1)
        self.k0 = torch.exp(logk) if logk is not None else torch.full_like(phi, ph.kmuf0)
        self.mn = torch.full_like(phi, ph.mu0)
        self.eta = torch.ones_like(phi)
        self.mus = self.mn * ph.phi0 * ph.cmu
        self.dts, self.cum, self.steps, self.first, self.it = ph.dtS, ph.dt, 0, True, 0

    # stresses: normal (zz, yy, xx) at the cells, shear on the edges
    def _maxwell(self, mu):
        xi = mu / (self.p.G * self.dts)
        return xi / (1.0 + xi), 2.0 * mu / (1.0 + xi)

    def _rates(self):
        e = [_dif(v, a) / self.d[a] for a, v in enumerate((self.vz, self.vy, self.vx))]
        return e, e[0] + e[1] + e[2]

    def _edge_mu(self, a, b):
        """Viscosity on the edges between axes a and b: the mean of the cells around, inside the domain."""
        m = _wall(_wall(self.mus, a), b)
        w = _wall(_wall(torch.ones_like(self.mus), a), b)
        return _avg(_avg(m, a), b) / _avg(_avg(w, a), b)

    def _shear(self, a, b, va, vb, so, bg=0.0):
        """a So + b e on the edges between axes a and b (va, vb: the velocities along them); zero on the walls
        (the background rate bg is added on every edge)."""
        e = 0.5 * (_dif(_inner(va, a), b) / self.d[b] + _dif(_inner(vb, b), a) / self.d[a])
        ca, cb = self._maxwell(self._edge_mu(a, b))
        rate = _wall(_wall(e, a), b) + bg
        if bg == 0.0:
            mask = _wall(_wall(torch.ones_like(e), a), b)
            return (ca * so + cb * rate) * mask
        return ca * so + cb * rate

    def _edges(self):
        return (self._shear(0, 1, self.vz, self.vy, self.syz), self._shear(0, 2, self.vz, self.vx, self.sxz),
                self._shear(1, 2, self.vy, self.vx, self.sxy, 0.5 * self.p.shear_bg))

    def begin_step(self, history):
        p = self.p
        if p.dts_rule:
            if self.steps >= 1:
                self.cum += p.dt
            new = float(self.mus.max()) / (p.G * p.xsi_w)
            history = self.steps >= 1 and self.cum >= new
        if history:
            e, div = self._rates()
            ca, cb = self._maxwell(self.mus)
            tau = [ca * s + cb * (x - div / 3.0) for s, x in zip(self.so, e)]
            self.syz, self.sxz, self.sxy = self._edges()
            self.so = tau
        if p.dts_rule:
            if history or self.steps == 0:
                self.cum = 0.0
            self.dts = new
        self.pto, self.pfo, self.lpo = self.pt, self.pf, self.lp
        self.steps += 1
        self.it = 0

    def refresh(self, r_eta, r_mu):
        p = self.p
        phi = 1.0 - torch.exp(self.lp)
        self.kc = self.k0 * (phi / p.phi0) ** 3
        eta = p.eta0 * self.mn * (p.phi0 / phi)
        eta = torch.where(self.pf > self.pt, eta / p.R0, eta)
        mn = torch.full_like(phi, p.mu0)
        if p.powerlaw or p.dpcap:
            e, div = self._rates()
            ca, cb = self._maxwell(self.mus)
            inv = sum((ca * s + cb * (x - div / 3.0)) ** 2 for s, x in zip(self.so, e)) * 0.5
            syz, sxz, sxy = self._edges()
            for t, a, b in ((syz, 0, 1), (sxz, 0, 2), (sxy, 1, 2)):
                inv += _avg(_avg(t, a), b) ** 2
            tii = torch.sqrt(inv)
            if p.powerlaw:
                mn = p.mu0 / (1.0 + (tii / p.tau0) ** (p.n_pow - 1.0))
            if p.dpcap:
                f = math.radians(p.fric_deg)
                cap = torch.clamp(p.coh * math.cos(f) + (self.pt - self.pf) * math.sin(f), min=p.tau_y_min)
                mn = torch.where(tii > 0.0, torch.minimum(mn, self.mn * cap / tii), mn)
        if not self.first:
            eta = torch.exp(r_eta * torch.log(eta) + (1.0 - r_eta) * torch.log(self.eta))
            mn = torch.exp(r_mu * torch.log(mn) + (1.0 - r_mu) * torch.log(self.mn))
        self.eta, self.mn, self.first = eta, mn, False
        self.mus = mn * p.phi0 * p.cmu

    def step(self, porosity):
        """One iteration; the residuals (momentum, Pt, Pf) of the state it starts from, as maxima, by call."""
        p, d = self.p, self.d
        h, nmax = min(d), max(self.n)
        s = torch.exp(self.lp)
        chi = 1.0 / (self.eta * s)
        e, div = self._rates()
        dtp = (1.0 + p.beta_n) / nmax * self.mus
        bd = p.beta_d / p.dt
        ptn = (self.pt - dtp * (div + bd * (-self.pto - p.alpha * (self.pf - self.pfo)) - self.pf * chi)) / (
            1.0 + dtp * (bd + chi))
        rpt = div + bd * ((self.pt - self.pto) - p.alpha * (self.pf - self.pfo)) + (self.pt - self.pf) * chi
        ca, cb = self._maxwell(self.mus)
        tau = [ca * so + cb * (x - div / 3.0 + p.beta_n * rpt) for so, x in zip(self.so, e)]
        syz, sxz, sxy = self._edges()
        # Darcy flux and fluid pressure
        rho_bg = p.rhofg * p.phi0 + (1.0 - p.phi0) * p.rhosg
        divq = torch.zeros_like(ptn)
        kl = self.kc.clone()
        for a in range(3):
            grad = _dif(self.pf, a) / d[a] + ((p.rhofg - rho_bg) if a == 0 else 0.0)
            divq += _dif(_wall(-_avg(self.kc, a) * grad, a), a) / d[a]
            n = self.n[a]
            lo, hi = self.kc.narrow(a, 0, n - 1), self.kc.narrow(a, 1, n - 1)
            kl.narrow(a, 1, n - 1).copy_(torch.maximum(kl.narrow(a, 1, n - 1), lo))
            kl.narrow(a, 0, n - 1).copy_(torch.maximum(kl.narrow(a, 0, n - 1), hi))
        dtf = h * h * (1.0 + p.beta_d * p.B / p.alpha) / p.c_pf / kl
        ab = p.alpha / p.B
        pfn = (self.pf - dtf * (divq + bd * (-ab * self.pfo - p.alpha * (self.pt - self.pto)) - self.pt * chi)) / (
            1.0 + dtf * (bd * ab + chi))
        rpf = divq + bd * (ab * (self.pf - self.pfo) - p.alpha * (self.pt - self.pto)) + (self.pf - self.pt) * chi
        # momentum
        rg = p.rhofg * (1.0 - s) + p.rhosg * s
        fz = (_dif(tau[0] - ptn, 0) / d[0] + _dif(_inner(syz, 0), 1) / d[1] + _dif(_inner(sxz, 0), 2) / d[2]
              - (_avg(rg, 0) - rho_bg))
        fy = _dif(tau[1] - ptn, 1) / d[1] + _dif(_inner(syz, 1), 0) / d[0] + _dif(_inner(sxy, 1), 2) / d[2]
        fx = _dif(tau[2] - ptn, 2) / d[2] + _dif(_inner(sxz, 2), 0) / d[0] + _dif(_inner(sxy, 2), 1) / d[1]
        w = cb * p.beta_n * rpt - ptn + self.pt
        def maxima():
            f = max(float((t - _dif(w, a) / d[a]).abs().max()) for a, t in enumerate((fz, fy, fx)) if t.numel())
            return f, max(float(rpt.abs().max()), float(rpf.abs().max()))
        if porosity:
            adv = torch.zeros_like(ptn)
            for a, v in enumerate((self.vz, self.vy, self.vx)):
                flux = 0.5 * _inner(v, a) * _dif(s, a) / d[a]
                adv += 2.0 * _avg(_wall(flux, a), a)
            rate = p.beta_phi * ((pfn - self.pfo) - (ptn - self.pto)) / p.dt + (pfn - ptn) / self.eta + adv
            self.lp = self.lpo - p.dt * rate
        c = p.rho_i * h * h / (p.c_v * (1.0 + p.beta_n))
        for a, (r, v, f) in enumerate((("rz", "vz", fz), ("ry", "vy", fy), ("rx", "vx", fx))):
            n = self.n[a]
            mu = torch.maximum(self.mus.narrow(a, 0, n - 1), self.mus.narrow(a, 1, n - 1))
            new = f / p.rho_i + (1.0 - p.damp_c / n) * getattr(self, r)
            setattr(self, r, new)
            setattr(self, v, getattr(self, v) + _wall(c / mu * new, a))
        self.pt, self.pf = ptn, pfn
        return maxima

    def iterate(self, n):
        for _ in range(n):
            if self.it % self.p.nup == 0:
                self.refresh(self.p.r_eta, self.p.r_mu)
            self.step(True)
            self.it += 1

    def solve(self, rtol):
        it, ref = 0, getattr(self, "ref", None)
        while True:
            it += 1
            maxima = self.step(False)
            if it % self.p.nup and not (it == 1 and ref is None):
                continue
            now = maxima()
            ref = self.ref = ref or now
            if it % self.p.nup == 0 and max(x / r for x, r in zip(now, ref) if r > 0) <= rtol:
                return

    def porosity_step(self):
        p, d = self.p, self.d
        s = torch.exp(self.lp)
        adv = torch.zeros_like(s)
        for a, v in enumerate((self.vz, self.vy, self.vx)):
            adv += 2.0 * _avg(_wall(0.5 * _inner(v, a) * _dif(s, a) / d[a], a), a)
        rate = p.beta_phi * ((self.pf - self.pfo) - (self.pt - self.pto)) / p.dt + (self.pf - self.pt) / self.eta + adv
        self.lp = self.lpo - p.dt * rate
