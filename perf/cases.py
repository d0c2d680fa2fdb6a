"""The work that users of the FDTD-PIC library have it do, as cases that can be timed and checked.

Four kinds of case, each through the Python entry points a program calls:

  step   a simulation that is kept: ``Simulation.step(n)``, then the new E and
         H read in place on the GPU (device_fields=True)
  run    a whole small run: build the simulation, step it, read fields,
         particles and probe spectra back, close it
  batch  a kept ``Batch`` of uneven simulations: ``Batch.step(n)``, then every
         member's E and H
  grad   a design loop's evaluation: ``spp_power`` forward and backward on
         float32 parameters that scale the Drude maps

Sizes, films, bunches and boundaries are those of the repository's workloads
(slab, production film, adjoint film, batched films, grating, the paper's
film) or lie between them.  A kept simulation goes on from pass to pass, so
the boxes are long enough (or periodic along the beam) for the bunch to stay
in them while a case is timed, and but for the grating, whose passes are few,
its charge is a tenth of the workloads' 1 fC, so that it does not blow apart.

``exact`` is the same scheme in FP64 in plain torch: the Yee updates with CPML,
the Drude current of Eq. 6, the trilinear gather, Boris push and Esirkepov
deposit, and the gradient by torch's own differentiation.
"""
import math
from types import SimpleNamespace

import numpy as np
import torch
from torch.utils.checkpoint import checkpoint

from paper_1505_04007_amd import native

C = 299792458.0
MU0 = 1.25663706212e-6
EPS0 = 1.0 / (MU0 * C * C)
ETA0 = MU0 * C
QE = 1.602176634e-19
ME = 9.1093837015e-31
WP = 1.37e16     # silver, rad/s
GAMMA = 3.2e13   # 1/s
BC = {"pec": native.BC_PEC, "periodic": native.BC_PERIODIC, "cpml": native.BC_CPML}


def _case(kind, nx, ny, nz, bc, **kw):
    c = {"kind": kind, "nx": nx, "ny": ny, "nz": nz, "bcx": bc[0], "bcy": bc[1], "bcz": bc[2],
         "npml": 8, "dx_nm": 2.0, "normal": "z", "film": 10, "groove": 0, "particles": 0,
         "kev": 50.0, "charge": 1e-16, "sx": 20.0, "sy": 5.0, "sz": 5.0, "gap_nm": 8.0, "steps": 20,
         "mode": 0, "tune": False, "members": 1, "ckpt": 0, "seeded_fields": False}
    c.update(kw)
    return c


OPEN = ("cpml", "cpml", "cpml")
WALLS = ("pec", "pec", "pec")


def listed():
    return [
        # the smallest call: one step of the 32^3 cavity, then a look at the fields
        # (interactive use, a coupled code that steps in lockstep): launches and latency
        dict(_case("step", 32, 32, 32, WALLS, npml=0, dx_nm=5.0, film=4, steps=1, seeded_fields=True),
             name="cavity32_step1"),
        # the smallest whole run, as a parity check or a parameter scan makes it:
        # build, 200 steps of the 1000-particle slab, read everything back
        dict(_case("run", 32, 32, 32, WALLS, npml=0, dx_nm=5.0, film=4, particles=1000, kev=30.0, charge=1e-15,
                   sx=5.0, gap_nm=0.0, steps=200), name="slab32_run200"),
        # the paper's own geometry: film normal along x, sheet bunch along z over
        # four periodic y cells, 2 nm cells, few particles
        dict(_case("step", 130, 4, 1700, ("cpml", "periodic", "cpml"), npml=10, normal="x", particles=4000,
                   kev=100.0, charge=1e-19, sx=2.0, sz=5.0, gap_nm=10.0, steps=50), name="paper20nm_2nm_step50"),
        # the same at 1 nm with one y cell and a long box, as the thickness sweep of
        # Table 1 runs it
        dict(_case("step", 281, 1, 3601, ("cpml", "periodic", "cpml"), npml=10, dx_nm=1.0, normal="x", film=60,
                   particles=4000, kev=100.0, charge=1e-19, sx=2.0, sz=5.0, gap_nm=10.0, steps=50),
             name="paper60nm_1nm_step50"),
        # fields only at an odd size: the film rings down in an open box with no bunch
        dict(_case("step", 301, 203, 157, OPEN, film=15, steps=10, seeded_fields=True), name="open_fields_odd"),
        # a film in a box periodic on all sides: a bunch train, reproducible
        # (fixed-point) deposit
        dict(_case("step", 96, 64, 96, ("periodic", "periodic", "periodic"), npml=0, particles=200_000, mode=2,
                   steps=20), name="train_fixed"),
        # one slab of a grating box, periodic along the beam: many particles on few cells
        dict(_case("step", 64, 128, 128, ("periodic", "cpml", "cpml"), npml=12, dx_nm=1.0, film=40, groove=10,
                   particles=1_000_000, kev=100.0, sx=20.0, sy=10.0, sz=10.0, gap_nm=5.0, steps=20),
             name="shard_periodic_x"),
        # the production film with its 1e6-particle bunch, a box long enough to keep it
        dict(_case("step", 448, 128, 128, OPEN, film=15, particles=1_000_000, steps=20), name="film_1e6"),
        # the largest: the grating run with 1e7 particles, tuned as the benchmark tunes it
        dict(_case("step", 512, 256, 256, OPEN, npml=12, dx_nm=1.0, film=40, groove=10, particles=10_000_000,
                   kev=100.0, charge=1e-15, sx=50.0, sy=10.0, sz=10.0, gap_nm=5.0, steps=20, tune=True),
             name="grating_1e7"),
        # a sweep over film thickness and energy: 16 uneven simulations together
        dict(_case("batch", 176, 64, 64, OPEN, particles=200_000, kev=35.0, steps=40, members=16), name="batch16"),
        # the gradient of the probe's spectral power, all snapshots kept
        dict(_case("grad", 128, 64, 64, OPEN, particles=100_000, charge=1e-15, steps=1000), name="grad_adjoint"),
        # the same on an odd box with checkpoints and replay
        dict(_case("grad", 91, 45, 53, ("cpml", "periodic", "cpml"), npml=6, film=6, particles=20_000, steps=300,
                   sx=10.0, ckpt=18), name="grad_checkpoints"),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["fields", "fields", "run", "paper", "paper", "train", "film", "film", "batch", "grad"])
    if kind == "fields":
        bc = tuple(rng.choice(["pec", "periodic", "cpml"]) for _ in range(3))
        return _case("step", _log_int(rng, 24, 400), _log_int(rng, 24, 200), _log_int(rng, 24, 200), bc,
                     npml=rng.randint(4, 11), film=rng.randint(3, 10), steps=rng.choice([1, 3, 10, 25]),
                     seeded_fields=True)
    if kind == "run":
        n = rng.randint(28, 44)
        return _case("run", n, n + rng.randint(0, 5), n + rng.randint(0, 5), WALLS, npml=0, dx_nm=5.0, film=4,
                     particles=_log_int(rng, 200, 20_000), kev=rng.uniform(20, 60), charge=1e-15, sx=5.0, gap_nm=0.0,
                     steps=rng.randint(50, 250))
    if kind == "paper":
        dx = rng.choice([1.0, 2.0])
        return _case("step", int(220 / dx) + rng.randint(0, 40), rng.choice([1, 1, 2, 4, 7]), rng.randint(1500, 3700),
                     ("cpml", "periodic", "cpml"), npml=10, dx_nm=dx, normal="x", film=rng.randint(10, 30),
                     particles=_log_int(rng, 1000, 20_000), kev=100.0, charge=1e-19, sx=2.0, sz=5.0, gap_nm=10.0,
                     steps=rng.randint(10, 60))
    if kind == "train":
        bc = ("periodic", rng.choice(["periodic", "cpml"]), rng.choice(["periodic", "cpml"]))
        return _case("step", rng.randint(48, 140), rng.randint(56, 130), rng.randint(72, 140), bc, npml=8,
                     particles=_log_int(rng, 20_000, 1_000_000), mode=rng.choice([0, 0, 2]), sx=10.0,
                     kev=rng.uniform(20, 100), steps=rng.randint(5, 30))
    if kind == "film":
        return _case("step", rng.randint(384, 470), rng.randint(60, 130), rng.randint(72, 130), OPEN,
                     npml=rng.randint(6, 12), film=rng.randint(5, 15), groove=rng.choice([0, 0, 4]),
                     particles=_log_int(rng, 20_000, 1_500_000), kev=rng.uniform(20, 60), steps=rng.randint(5, 30))
    if kind == "batch":
        return _case("batch", 16 * rng.randint(10, 12), 16 * rng.randint(3, 5), 16 * rng.randint(4, 5), OPEN,
                     particles=_log_int(rng, 20_000, 150_000), kev=rng.uniform(20, 40), steps=rng.randint(20, 50),
                     members=rng.randint(3, 9))
    bc = ("cpml", rng.choice(["cpml", "periodic"]), "cpml")
    return _case("grad", rng.randint(72, 128), rng.randint(44, 64), rng.randint(52, 64), bc, npml=rng.randint(5, 8),
                 film=rng.randint(5, 10), particles=_log_int(rng, 5_000, 100_000), sx=10.0, steps=rng.randint(150, 600),
                 ckpt=rng.choice([0, 0, 20]))


# ---------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------

def _grid(case):
    n = (case["nx"], case["ny"], case["nz"])
    dx = case["dx_nm"] * 1e-9
    return n, dx, 0.5 * dx / (C * math.sqrt(3.0)), (case["bcx"], case["bcy"], case["bcz"])


def _film_span(case):
    """First and last + 1 cell of the film along its normal."""
    if case["normal"] == "x":
        lo = (case["nx"] - case["film"]) // 2
        return lo, lo + case["film"]
    top = case["nz"] // 2
    return top - case["film"], top


def _maps(case):
    """Relative Drude maps (1 in the metal, 0 in vacuum), (nx, ny, nz), x fastest in memory."""
    n, dx, _, _ = _grid(case)
    m = np.zeros(n[::-1]).transpose(2, 1, 0)
    lo, hi = _film_span(case)
    if case["normal"] == "x":
        m[lo:hi] = 1.0
    else:
        m[:, :, lo:hi] = 1.0
        if case["groove"]:
            cut = np.mod((np.arange(n[0]) + 0.5) * dx, 100e-9) >= 50e-9
            m[cut, :, hi - case["groove"]:hi] = 0.0
    return m


def _normal(rng, n):
    """Standard normal values, those beyond 3 drawn again."""
    g = rng.standard_normal(n)
    while True:
        bad = np.nonzero(np.abs(g) > 3.0)[0]
        if not bad.size:
            return g
        g[bad] = rng.standard_normal(bad.size)


def _bunch(case, seed):
    """A cold Gaussian bunch gliding gap_nm above the film (its lower edge), along +x, or
    along +z over a film whose normal is x (then uniform in y); None without particles."""
    np_ = case["particles"]
    if not np_:
        return None
    rng = np.random.default_rng([150504007, seed])
    n, dx, _, bc = _grid(case)
    L = [q * dx for q in n]
    g = 1.0 + case["kev"] * 1e3 * QE / (ME * C * C)
    u = C * math.sqrt(g * g - 1.0)
    s = [case["sx"] * 1e-9, case["sy"] * 1e-9, case["sz"] * 1e-9]
    top = _film_span(case)[1] * dx
    pml = case["npml"] * dx if bc[2 if case["normal"] == "x" else 0] == "cpml" else dx
    if case["normal"] == "x":
        x = top + case["gap_nm"] * 1e-9 + s[0] * _normal(rng, np_)
        y = rng.uniform(0.0, L[1], np_)
        z = pml + 12 * dx + 3 * s[2] + s[2] * _normal(rng, np_)
        u3 = (0.0, 0.0, u)
    else:
        x = pml + 3 * s[0] + s[0] * _normal(rng, np_)
        y = 0.5 * L[1] + s[1] * _normal(rng, np_)
        z = top + case["gap_nm"] * 1e-9 + 3 * s[2] + s[2] * _normal(rng, np_)
        u3 = (u, 0.0, 0.0)
    pos = []
    for q, per, length in zip((x, y, z), bc, L):
        pos.append(np.mod(q, length) if per == "periodic" else np.clip(q, 1e-3 * dx, length - 1e-3 * dx))
    return SimpleNamespace(x=pos[0], y=pos[1], z=pos[2], ux=np.full(np_, u3[0]), uy=np.full(np_, u3[1]),
                           uz=np.full(np_, u3[2]), n=np_, q=-QE, m=ME, w=case["charge"] / (np_ * QE))


def _init_E(case, seed):
    """Two smooth pulses of seeded place, width and direction in each component of E (nx, ny, nz), or None."""
    if not case["seeded_fields"]:
        return None
    rng = np.random.default_rng([150504008, seed])
    n, _, _, _ = _grid(case)
    pulses = [(rng.uniform(0.3, 0.7, 3), rng.uniform(2.0, 4.0), 1e6 * rng.standard_normal(3)) for _ in range(2)]
    out = []
    for c in range(3):
        e = np.zeros(n[::-1])
        for at, width, amp in pulses:
            ax = [np.exp(-(np.arange(n[d]) + (0.5 if d == c else 0.0) - at[d] * n[d]) ** 2 / (2 * width ** 2))
                  for d in range(3)]
            e += amp[c] * ax[2][:, None, None] * ax[1][None, :, None] * ax[0][None, None, :]
        out.append(e.transpose(2, 1, 0))
    return out


def _probes(case):
    n, dx, _, _ = _grid(case)
    top = _film_span(case)[1] * dx
    if case["normal"] == "x":
        return np.array([[top + 1e-9, (n[1] // 2) * dx, f * n[2] * dx] for f in (0.4, 0.8)])
    return np.array([[f * n[0] * dx, 0.5 * n[1] * dx, top + 1.1 * dx] for f in (0.5, 0.625, 0.75)])


def _omegas(case):
    return WP * np.linspace(0.3, 1.0, 64)


def _simulation(case, seed, wp, gamma, **kw):
    n, dx, dt, bc = _grid(case)
    return native.Simulation(*n, dx, dt, wp, gamma, bc=[BC[b] for b in bc], npml=case["npml"], bunch=_bunch(case, seed),
                             probes=_probes(case), omega=_omegas(case), sort_every=20, init_E=_init_E(case, seed),
                             deposit_mode=case["mode"], **kw)


def _member(case, i):
    """Member i of a batch: film, box and energy grow with i."""
    f = i / max(case["members"] - 1, 1)
    g = 1.0 + 0.4 * f
    return dict(case, kind="step", members=1, nx=16 * round(case["nx"] * g / 16), ny=16 * round(case["ny"] * g / 16),
                nz=16 * round(case["nz"] * g / 16), film=3 + round(25 * f), kev=case["kev"] * (0.6 + 0.8 * f))


def _omega0(case):
    return 0.68 * WP


def _scales(case, seed):
    """The design parameters of a gradient case: relative Drude maps with 5 % seeded noise, float32 on the GPU."""
    rng = np.random.default_rng([150504009, seed])
    m = _maps(case)
    out = []
    for _ in range(2):
        t = np.where(m > 0, 1.0 + 0.05 * np.clip(rng.standard_normal(m.shape), -3, 3), 0.0)
        out.append(torch.from_numpy(t).float().to("cuda"))
    return out


def prepare(case, seed):
    kind = case["kind"]
    if kind == "batch":
        sims = []
        for i in range(case["members"]):
            c = _member(case, i)
            m = _maps(c)
            sims.append(_simulation(c, seed + 1000 * (i + 1), WP * m, GAMMA * m, device_fields=True))
        return SimpleNamespace(case=case, batch=native.Batch(sims, use_graph=True), sims=sims)
    if kind == "grad":
        n, dx, dt, bc = _grid(case)
        bunch = _bunch(case, seed)

        def make_sim(wp, gamma):
            return native.Simulation(*n, dx, dt, wp, gamma, bc=[BC[b] for b in bc], npml=case["npml"], bunch=bunch,
                                     probes=_probes(case), omega=np.array([_omega0(case)]), sort_every=20,
                                     deposit_mode=case["mode"])

        return SimpleNamespace(case=case, scales=_scales(case, seed),
                               power=native.spp_power(make_sim, _omega0(case), case["steps"], case["ckpt"]))
    m = _maps(case)
    if kind == "run":
        return SimpleNamespace(case=case, seed=seed, wp=WP * m, gamma=GAMMA * m)
    sim = _simulation(case, seed, WP * m, GAMMA * m, device_fields=True)
    if case["tune"]:
        sim.tune(reps=10)
    return SimpleNamespace(case=case, sim=sim)


def run(state):
    case = state.case
    kind = case["kind"]
    if kind == "step":
        state.sim.step(case["steps"])
        return {"E": state.sim.device_E(), "H": state.sim.device_H()}
    if kind == "batch":
        state.batch.step(case["steps"])
        return {"E": [s.device_E() for s in state.sims], "H": [s.device_H() for s in state.sims]}
    if kind == "run":
        sim = _simulation(case, state.seed, state.wp, state.gamma)
        sim.step(case["steps"])
        # the state is held in 32 bits, and saved as such
        out = {"E": sim.fields(native.FIELD_E).astype(np.float32), "H": sim.fields(native.FIELD_H).astype(np.float32),
               "particles": sim.particles().astype(np.float32), "spectra": sim.probe().astype(np.complex64)}
        sim.close()
        return out
    s, t = (q.detach().requires_grad_() for q in state.scales)
    loss = torch.log(state.power(WP * s.double(), GAMMA * t.double())).to(s.dtype)
    loss.backward()
    return {"loss": loss.detach(), "ds": s.grad, "dt": t.grad}


def work(case):
    if case["kind"] == "batch":
        parts = [work(_member(case, i)) for i in range(case["members"])]
        return {k: sum(p[k] for p in parts) for k in ("bytes", "flops")}
    n, _, _, bc = _grid(case)
    cells = n[0] * n[1] * n[2]
    slab = sum(2 * case["npml"] * cells / n[a] for a in range(3) if bc[a] == "cpml")
    metal = cells * case["film"] / (n[0] if case["normal"] == "x" else n[2])
    # a step: E and H read and written once, the CPML memories of E and H of the
    # layer cells, the Drude current and its coefficients, the particles
    b = 48 * cells + 32 * slab + 32 * metal + 48 * case["particles"]
    f = 36 * cells + 16 * slab + 15 * metal + 700 * case["particles"]
    if case["kind"] == "grad":
        # the run, and the transposed step back through it with the metal's snapshots written and read
        b = 2 * b - 48 * case["particles"] + 48 * metal
        f = 2 * f - 700 * case["particles"] + 30 * metal
    return {"bytes": float(b * case["steps"]), "flops": float(f * case["steps"])}


# ---------------------------------------------------------------------------
# the scheme in FP64, plain torch
# ---------------------------------------------------------------------------

def _dev():
    return torch.device("cuda" if torch.cuda.is_available() else "cpu")


class _Exact:
    """FP64 state of one simulation: arrays (nz, ny, nx), E in V/m, H times eta0, J times dt/eps0."""

    def __init__(self, case, seed, wp, gamma, probes=None):
        self.n, self.dx, self.dt, bc = _grid(case)
        self.case, self.dev = case, _dev()
        self.per = [b == "periodic" for b in bc]
        self.S = C * self.dt / self.dx
        shape = self.n[::-1]
        z = lambda: torch.zeros(shape, dtype=torch.float64, device=self.dev)  # noqa: E731
        self.E, self.H, self.J = [z() for _ in range(3)], [z() for _ in range(3)], [z() for _ in range(3)]
        self.coef(wp, gamma)
        # CPML: per axis (b, c, 1/kappa) at nodes (E) and half nodes (H), and the memories
        self.pml, self.psiE, self.psiH = [], [], []
        for a in range(3):
            on = bc[a] == "cpml"
            self.pml.append([self._layer(a, off) for off in (0.0, 0.5)] if on else None)
            self.psiE.append([z(), z()] if on else [None, None])
            self.psiH.append([z(), z()] if on else [None, None])
        # tangential E on the stored walls stays 0
        self.mask = []
        for c in range(3):
            m = torch.ones(shape, dtype=torch.float64, device=self.dev)
            for a in range(3):
                if a != c and not self.per[a]:
                    m.select(2 - a, 0).zero_()
            self.mask.append(m)
        init = _init_E(case, seed)
        if init is not None:
            for c in range(3):
                self.E[c] = self.mask[c] * torch.from_numpy(np.ascontiguousarray(init[c].transpose(2, 1, 0))).to(self.dev)
        b = _bunch(case, seed)
        self.b = b
        if b is not None:
            t = lambda v, s: torch.from_numpy(v).to(self.dev) / s  # noqa: E731
            self.x = [t(b.x, self.dx), t(b.y, self.dx), t(b.z, self.dx)]
            self.u = [t(b.ux, C), t(b.uy, C), t(b.uz, C)]
            self.live = torch.ones(b.n, dtype=torch.bool, device=self.dev)
        self.step = 0

    def coef(self, wp, gamma):
        den = 2.0 + gamma * self.dt
        self.cb, self.d = 2.0 * (wp * self.dt) ** 2 / den, 2.0 * gamma * self.dt / den

    def _layer(self, a, off):
        n, L = self.n[a], float(self.case["npml"])
        pos = np.arange(n) + off
        r = np.clip(np.maximum(L - pos, pos - (n - L)), 0.0, None) / L
        sig = 0.8 * 4.0 / (ETA0 * self.dx) * r ** 3
        b = np.exp(-sig * self.dt / EPS0)
        view = [1, 1, 1]
        view[2 - a] = n
        return [torch.from_numpy(v).to(self.dev).reshape(view) for v in (b, np.where(sig > 0, b - 1.0, 0.0))]

    def _diff(self, f, a, d):
        """f at the next node along axis a minus f (d = 1), or f minus the one before (d = -1); 0 beyond a wall."""
        dim, n = 2 - a, self.n[a]
        if d > 0:
            edge = f.narrow(dim, 0, 1) if self.per[a] else torch.zeros_like(f.narrow(dim, 0, 1))
            return torch.cat([f.narrow(dim, 1, n - 1), edge], dim) - f
        edge = f.narrow(dim, n - 1, 1) if self.per[a] else torch.zeros_like(f.narrow(dim, 0, 1))
        return f - torch.cat([edge, f.narrow(dim, 0, n - 1)], dim)

    # the two components whose curls differentiate along axis a, and the component they read
    def _curl(self, F, psi, off, d):
        """curl of F by one-sided differences (d = +1 or -1) with the layers' stretching; new memories."""
        out, new = [0.0, 0.0, 0.0], [[None, None] for _ in range(3)]
        for c in range(3):
            for a, r, s in (((c + 1) % 3, (c + 2) % 3, 1.0), ((c + 2) % 3, (c + 1) % 3, -1.0)):
                g = self._diff(F[r], a, d)
                if self.pml[a] is not None:
                    q = sorted({0, 1, 2} - {a}).index(c)
                    b, k = self.pml[a][off]
                    new[a][q] = b * psi[a][q] + k * g
                    g = g + new[a][q]
                out[c] = out[c] + s * g
        return out, new

    def h_update(self, st):
        E, H, J, psiE, psiH = st
        curl, psiH = self._curl(E, psiH, 1, 1)
        return E, [H[c] - self.S * curl[c] for c in range(3)], J, psiE, psiH

    def e_update(self, st, Jb):
        E, H, J, psiE, psiH = st
        J = [J[c] + self.cb * E[c] - self.d * J[c] for c in range(3)]
        curl, psiE = self._curl(H, psiE, 0, -1)
        E = [E[c] + self.mask[c] * (self.S * curl[c] - J[c] - (Jb[c] if Jb is not None else 0.0)) for c in range(3)]
        return E, H, J, psiE, psiH

    def state(self):
        return self.E, self.H, self.J, self.psiE, self.psiH

    def keep(self, st):
        self.E, self.H, self.J, self.psiE, self.psiH = st

    def _gather(self, F, half):
        """Trilinear value at the particles of a component at half nodes along the axes in `half`."""
        ix, wt = [], []
        for a in range(3):
            s = self.x[a] - (0.5 if half[a] else 0.0)
            f = torch.floor(s)
            i, w = f.long(), s - f
            pair = []
            for k, wk in ((i, 1.0 - w), (i + 1, w)):
                if self.per[a]:
                    pair.append((k % self.n[a], wk))
                else:
                    pair.append((k.clamp(0, self.n[a] - 1), wk * ((k >= 0) & (k < self.n[a]))))
            ix.append([p[0] for p in pair])
            wt.append([p[1] for p in pair])
        v, flat = 0.0, F.reshape(-1)
        for c in range(2):
            for b in range(2):
                for q in range(2):
                    at = ix[0][q] + self.n[0] * (ix[1][b] + self.n[1] * ix[2][c])
                    v = v + wt[0][q] * wt[1][b] * wt[2][c] * flat[at]
        return v

    def push(self, Hold):
        """Gather, Boris, move; returns the deposited current of the three components."""
        B = [0.5 * (Hold[c] + self.H[c]) for c in range(3)]
        ah = self.b.q * self.dt / (2.0 * self.b.m * C)
        e = [ah * self._gather(self.E[c], [a == c for a in range(3)]) for c in range(3)]
        h = [ah * self._gather(B[c], [a != c for a in range(3)]) for c in range(3)]
        m = [self.u[c] + e[c] for c in range(3)]
        g = 1.0 / torch.sqrt(1.0 + m[0] ** 2 + m[1] ** 2 + m[2] ** 2)
        t = [v * g for v in h]
        f = 2.0 / (1.0 + t[0] ** 2 + t[1] ** 2 + t[2] ** 2)
        cross = lambda p, q: [p[1] * q[2] - p[2] * q[1], p[2] * q[0] - p[0] * q[2], p[0] * q[1] - p[1] * q[0]]  # noqa: E731
        w = cross(m, t)
        w = cross([m[c] + w[c] for c in range(3)], [f * t[c] for c in range(3)])
        u = [torch.where(self.live, m[c] + w[c] + e[c], self.u[c]) for c in range(3)]
        g = 1.0 / torch.sqrt(1.0 + u[0] ** 2 + u[1] ** 2 + u[2] ** 2)
        x0, x1, dep = self.x, [self.x[c] + self.S * u[c] * g for c in range(3)], self.live.clone()
        for a in range(3):
            if not self.per[a]:
                dep &= (x1[a] >= 0) & (x1[a] < self.n[a])
        x1 = [torch.where(dep, x1[c], x0[c]) for c in range(3)]
        Jb = self._deposit(x0, x1)
        self.u, self.live = u, dep
        self.x = [torch.remainder(x1[c], float(self.n[c])) if self.per[c] else x1[c] for c in range(3)]
        return Jb

    def _deposit(self, x0, x1):
        """Esirkepov's current of first-order shapes on the three nodes each move touches."""
        base = [torch.minimum(torch.floor(p), torch.floor(q)).long() for p, q in zip(x0, x1)]
        S0, D, at, ok = [], [], [], []
        for a in range(3):
            r0, r1 = x0[a] - base[a], x1[a] - base[a]
            s0 = [torch.clamp(1.0 - (r0 - m).abs(), min=0.0) for m in range(3)]
            s1 = [torch.clamp(1.0 - (r1 - m).abs(), min=0.0) for m in range(3)]
            S0.append(s0)
            D.append([p - q for p, q in zip(s1, s0)])
            k = [base[a] + m for m in range(3)]
            at.append([v % self.n[a] if self.per[a] else v.clamp(0, self.n[a] - 1) for v in k])
            ok.append([torch.ones_like(v, dtype=torch.float64) if self.per[a] else
                       ((v >= 0) & (v < self.n[a])).double() for v in k])
        qd = -self.b.q * self.b.w / (EPS0 * self.dx ** 2)
        J = [torch.zeros(self.n[::-1], dtype=torch.float64, device=self.dev).reshape(-1) for _ in range(3)]
        for c in range(3):
            a, b = (c + 1) % 3, (c + 2) % 3
            for m in range(2):
                run = D[c][0] if m == 0 else D[c][0] + D[c][1]
                for p in range(3):
                    for q in range(3):
                        T = (S0[a][p] * S0[b][q] + 0.5 * (D[a][p] * S0[b][q] + S0[a][p] * D[b][q]) +
                             D[a][p] * D[b][q] / 3.0)
                        k = {c: m, a: p, b: q}
                        v = qd * run * T * ok[0][k[0]] * ok[1][k[1]] * ok[2][k[2]]
                        J[c].index_add_(0, at[0][k[0]] + self.n[0] * (at[1][k[1]] + self.n[1] * at[2][k[2]]), v)
        return [j.reshape(self.n[::-1]) for j in J]

    def advance(self, steps, each=None):
        for _ in range(steps):
            Hold = self.H
            self.keep(self.h_update(self.state()))
            Jb = self.push(Hold) if self.b is not None else None
            self.keep(self.e_update(self.state(), Jb))
            self.step += 1
            if each is not None:
                each(self, Jb)

    def probe_index(self):
        idx = []
        for p in _probes(self.case) / self.dx:
            i, j, k = math.floor(p[0] + 0.5), math.floor(p[1] + 0.5), math.floor(p[2])
            idx.append(i + self.n[0] * (j + self.n[1] * k))
        return torch.tensor(idx, device=self.dev)


def _exact_of(case, seed, scales=None):
    if scales is None:
        m = torch.from_numpy(np.ascontiguousarray(_maps(case).transpose(2, 1, 0))).to(_dev())
        return _Exact(case, seed, WP * m, GAMMA * m)
    s, t = (q.double().to(_dev()).permute(2, 1, 0) for q in scales)
    return _Exact(case, seed, WP * s, GAMMA * t)


def _stacked(x):
    return {"E": torch.stack(x.E), "H": torch.stack(x.H)}


def _exact_run(case, seed):
    x = _exact_of(case, seed)
    om = torch.from_numpy(_omegas(case)).to(x.dev)
    idx = x.probe_index()
    F = torch.zeros(len(idx), len(om), dtype=torch.complex128, device=x.dev)

    def sample(x, _):
        F.add_(x.dt * x.E[2].reshape(-1)[idx][:, None] * torch.exp(-1j * om * (x.step * x.dt))[None, :])

    x.advance(case["steps"], sample)
    gone = torch.full_like(x.x[0], math.nan)
    part = [torch.where(x.live, v * x.dx, gone) for v in x.x] + [v * C for v in x.u]
    xyz = lambda F, s: torch.stack([f.permute(2, 1, 0) * s for f in F]).contiguous().cpu().numpy()  # noqa: E731
    return {"E": xyz(x.E, 1.0), "H": xyz(x.H, 1.0 / ETA0), "particles": torch.stack(part).cpu().numpy(),
            "spectra": F.cpu().numpy()}


def _exact_grad(case, seed):
    """The bunch current of a forward run, then torch's derivative of the run with that current prescribed."""
    scales = _scales(case, seed)
    x = _exact_of(case, seed, scales)
    rec = []
    with torch.no_grad():
        x.advance(case["steps"], lambda x, Jb: rec.append(Jb))
    y = _exact_of(case, seed, scales)
    s, t = (q.double().to(y.dev).requires_grad_() for q in scales)
    idx = y.probe_index()
    layers = [a for a in range(3) if y.pml[a] is not None]

    def pack(st):
        E, H, J, pE, pH = st
        return [*E, *H, *J] + [pE[a][q] for a in layers for q in range(2)] + [pH[a][q] for a in layers for q in range(2)]

    def unpack(v):
        pE, pH = [[None, None] for _ in range(3)], [[None, None] for _ in range(3)]
        for k, a in enumerate(layers):
            pE[a] = list(v[9 + 2 * k:11 + 2 * k])
            pH[a] = list(v[9 + 2 * (len(layers) + k):11 + 2 * (len(layers) + k)])
        return list(v[0:3]), list(v[3:6]), list(v[6:9]), pE, pH

    def segment(first, count, wp, gamma, *v):
        y.coef(wp, gamma)
        st, ez = unpack(v), []
        for r in range(first, first + count):
            st = y.e_update(y.h_update(st), rec[r])
            ez.append(st[0][2].reshape(-1)[idx])
        return (torch.stack(ez), *pack(st))

    wp, gamma = WP * s.permute(2, 1, 0), GAMMA * t.permute(2, 1, 0)
    v, ez = pack(y.state()), []
    for first in range(0, case["steps"], 25):
        out = checkpoint(segment, first, min(25, case["steps"] - first), wp, gamma, *v, use_reentrant=False)
        ez.append(out[0])
        v = out[1:]
    ez = torch.cat(ez)
    ph = _omega0(case) * y.dt * torch.arange(1, case["steps"] + 1, dtype=torch.float64, device=y.dev)[:, None]
    re, im = (y.dt * ez * torch.cos(ph)).sum(0), (y.dt * ez * torch.sin(ph)).sum(0)
    loss = torch.log((re ** 2 + im ** 2).sum())
    loss.backward()
    metal = [(q > 0).double().to(y.dev) for q in scales]
    return {"loss": loss.detach(), "ds": s.grad * metal[0], "dt": t.grad * metal[0]}


def exact(case, seed):
    if case["kind"] == "grad":
        return _exact_grad(case, seed)
    with torch.no_grad():
        if case["kind"] == "run":
            return _exact_run(case, seed)
        if case["kind"] == "batch":
            got = []
            for i in range(case["members"]):
                x = _exact_of(_member(case, i), seed + 1000 * (i + 1))
                x.advance(case["steps"])
                got.append(_stacked(x))
                del x
            return {k: [g[k] for g in got] for k in ("E", "H")}
        x = _exact_of(case, seed)
        x.advance(case["steps"])
        return _stacked(x)
