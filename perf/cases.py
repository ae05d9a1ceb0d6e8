"""The work that a user of this package has it do, as cases that can be timed
and compared: time steps of one packet (small to large grids, both precisions,
every kind of field and boundary), steps of a batch of packets, the gradient
of a final observable, and the eigenvalue modes of both discretisations.

A case is a dict of plain values.  `prepare` makes its inputs on the GPU from
the seed, `run` is one pass through the package's public classes and
functions, `exact` the same result from plain torch and numpy in 64 bits
(time steps by a Chebyshev expansion of exp(-i dt H), eigenvalues by a Lanczos
recurrence of its own).
"""
from __future__ import annotations

import math

import numpy as np
import torch
from torch.utils.checkpoint import checkpoint

from paper_1407_7370_amd import binding
from paper_1407_7370_amd.packets import C_LIGHT

MC2 = C_LIGHT * C_LIGHT
PI = math.pi


def _step(name, nx, ny, half_x, half_y, m, dt, steps, precision, **kw):
    """A packet of width sigma on the box [-half, half)^2, `steps` steps."""
    c = dict(name=name, kind="step", nx=nx, ny=ny, half_x=half_x, half_y=half_y, m=m, dt=dt, steps=steps,
             precision=precision, bc_x=0, bc_y=0, bz=0.0, pot_kind=0, pot_z=0.0, pot_a=0.0, chirality=1,
             pulse="none", a0=0.0, t_pulse=1.0, harmonics=0, sigma=2.0, p_max=0.0, p_x=0.0, spread=0.0,
             tuned=False)
    c.update(kw)
    return c


def listed():
    return [
        # the smallest grid in use: many short steps, bound by latency and launches
        _step("free-64", 64, 64, 20.0, 20.0, 10, 1e-3, 20, "fp64", bc_x=1, bc_y=1, p_max=50.0),
        # pulse shaping: a grid that one optimisation loop steps thousands of times
        _step("fourier-512", 512, 512, 20.0, 20.0, 12, 1e-3, 20, "fp64", pulse="fourier", harmonics=4, a0=20.0,
              t_pulse=2.0, p_max=50.0, tuned=True),
        # a ragged rectangle with every term of the Hamiltonian and mixed boundaries
        _step("ragged-1001x777", 1001, 777, 39.0, 30.0, 13, 4e-4, 6, "mixed", bc_x=1, bz=0.3, pot_kind=2, pot_z=1.5,
              chirality=-1, pulse="sin", a0=20.0, t_pulse=0.05, sigma=2.5, p_max=10.0),
        # bound states in a magnetic field: an ordinary grid, long Krylov spaces
        _step("landau-1024", 1024, 1024, 40.0, 40.0, 20, 5e-4, 5, "fp64", bz=0.5, pot_kind=1, pot_z=1.0, pot_a=1.0,
              sigma=3.0, spread=1.0),
        # the workload of the package's benchmark, in both precisions
        _step("laser-4096-mixed", 4096, 4096, 40.0, 40.0, 16, 2e-4, 4, "mixed", pulse="sin", a0=50.0, t_pulse=0.1,
              sigma=3.0, p_max=50.0, tuned=True),
        _step("laser-4096-fp64", 4096, 4096, 40.0, 40.0, 16, 2e-4, 4, "fp64", pulse="sin", a0=50.0, t_pulse=0.1,
              sigma=3.0, p_max=50.0, tuned=True),
        # the largest grid: the wave packet of the paper's own scaling runs
        _step("paper-8192", 8192, 8192, 0.02, 0.02, 10, 1e-7, 2, "fp64", bc_x=1, bc_y=1, sigma=1.0 / 800.0, p_x=100.0),
        # an ensemble: packets of mixed sizes and fields stepped together
        dict(name="batch-128", kind="batch", packets=128, n_min=128, n_max=512, h=0.078125, m=12, dt=3e-4, steps=4,
             precision="mixed"),
        # one evaluation of an optimisation loop over the pulse: loss and gradient
        dict(name="adjoint-512", kind="adjoint", n=512, half=20.0, m=12, dt=1e-3, steps=100, every=50, harmonics=4,
             a0=20.0, t_pulse=2.0, sigma=2.0, p_max=50.0, loss=9),
        # the lowest levels in a window by the plain recurrence
        dict(name="levels-1024", kind="levels", nx=1024, ny=1024, half=40.0, bz=0.5, pot_z=1.0, k_max=2000, wanted=4,
             above=5.0, tol=1e-6),
        # levels with their states: full reorthogonalisation
        dict(name="states-256", kind="states", nx=256, ny=256, half=20.0, bz=0.5, pot_z=1.0, k_max=512, wanted=2,
             above=2.0, tol=1e-6),
        # a scan of ground states in the pseudospectral discretisation
        dict(name="hermite-256", kind="hermite", problems=256, n=64, z_min=1.0, z_max=50.0, bz=0.0, k_max=1000,
             tol=2.5e-6),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _draw_step(rng):
    nx = _log_int(rng, 48, 4096)
    ny = max(48, min(4096, int(nx * math.exp(rng.uniform(-0.7, 0.7)))))
    h = math.exp(rng.uniform(math.log(0.02), math.log(0.3)))
    m = rng.randint(8, 20)
    norm = math.hypot(MC2, C_LIGHT * math.sqrt(2.0) / h)  # of the free lattice Hamiltonian
    precision = rng.choice(["mixed", "fp64"])
    # complex64 vectors are for short steps: their rounding grows with dt
    dt = m * math.exp(rng.uniform(math.log(0.15), math.log(0.35 if precision == "mixed" else 1.2))) / norm
    steps = max(1, min(20, int(6e7 / (nx * ny * m))))
    c = _step("", nx, ny, 0.5 * nx * h, 0.5 * ny * h, m, dt, steps, precision,
              bc_x=rng.randint(0, 1), bc_y=rng.randint(0, 1), sigma=max(0.04 * min(nx, ny) * h, 3.0 * h),
              p_max=min(50.0, 0.3 / h), chirality=rng.choice([1, -1]))
    if rng.random() < 0.4:
        c.update(bz=rng.uniform(0.1, 1.0), bc_x=0, bc_y=0)
    if rng.random() < 0.4:
        c.update(pot_kind=rng.choice([1, 2]), pot_z=rng.uniform(0.5, 3.0), pot_a=rng.uniform(0.5, 1.5))
    pulse = rng.choice(["none", "sin", "fourier"])
    if pulse != "none":
        c.update(pulse=pulse, a0=rng.uniform(5.0, 40.0), t_pulse=dt * rng.uniform(5.0, 200.0),
                 harmonics=4 if pulse == "fourier" else 0)
    del c["name"]
    return c


def draw(rng):
    """One more case of the listed ranges, sizes spread over their logarithm."""
    u = rng.random()
    if u < 0.55:
        return _draw_step(rng)
    if u < 0.70:
        n_min = rng.randint(90, 200)
        return dict(kind="batch", packets=_log_int(rng, 8, 128), n_min=n_min, n_max=rng.randint(n_min + 20, 512),
                    h=rng.uniform(0.05, 0.1), m=rng.randint(8, 14), dt=rng.uniform(1e-4, 3e-4), steps=rng.randint(1, 4),
                    precision=rng.choice(["mixed", "fp64"]))
    if u < 0.80:
        n = _log_int(rng, 64, 512)
        return dict(kind="adjoint", n=n, half=20.0, m=rng.randint(10, 14), dt=rng.uniform(4e-4, 1e-3),
                    steps=rng.randint(20, 100), every=rng.randint(10, 50), harmonics=4, a0=rng.uniform(5.0, 20.0),
                    t_pulse=2.0, sigma=2.0, p_max=min(50.0, 0.3 * n / 40.0), loss=9)
    if u < 0.90:
        nx = _log_int(rng, 160, 1024)
        return dict(kind="levels", nx=nx, ny=nx + rng.randint(-30, 30), half=40.0, bz=rng.uniform(0.4, 0.6), pot_z=1.0,
                    k_max=2000, wanted=rng.randint(2, 5), above=5.0, tol=1e-6)
    return dict(kind="hermite", problems=_log_int(rng, 1, 256), n=rng.choice([32, 48, 64]), z_min=rng.uniform(1.0, 5.0),
                z_max=rng.uniform(10.0, 50.0), bz=rng.choice([0.0, rng.uniform(0.001, 0.02)]), k_max=1000, tol=2.5e-6)


# ---------------------------------------------------------------------------
# Inputs
# ---------------------------------------------------------------------------
def _problem(c, coef=None):
    """The package's problem dict of a step case."""
    return dict(nx=c["nx"], ny=c["ny"], x_min=-c["half_x"], x_max=c["half_x"], y_min=-c["half_y"], y_max=c["half_y"],
                bc_x=c["bc_x"], bc_y=c["bc_y"], mass=1.0, c=C_LIGHT, charge=-1.0, bz=c["bz"], pot_kind=c["pot_kind"],
                pot_z=c["pot_z"], pot_a=c["pot_a"], chirality=c["chirality"],
                pulse_kind={"none": 0, "sin": 1, "fourier": 2}[c["pulse"]], pulse_e=(0.0, 1.0),
                a0=c["a0"] if c["pulse"] == "sin" else 0.0, omega=1.0 if c["pulse"] == "sin" else 0.0,
                t_pulse=c["t_pulse"], coef=coef)


def _axes(prob):
    x = prob["x_min"] + (prob["x_max"] - prob["x_min"]) / prob["nx"] * torch.arange(prob["nx"], dtype=torch.float64,
                                                                                   device="cuda")
    y = prob["y_min"] + (prob["y_max"] - prob["y_min"]) / prob["ny"] * torch.arange(prob["ny"], dtype=torch.float64,
                                                                                   device="cuda")
    return x, y, (prob["x_max"] - prob["x_min"]) / prob["nx"], (prob["y_max"] - prob["y_min"]) / prob["ny"]


def _dft(n, sign):
    """Matrix of the discrete Fourier transform of n points."""
    j = torch.arange(n, dtype=torch.int64, device="cuda")
    ph = (sign * 2 * PI / n) * (j[:, None] * j[None, :] % n).double()
    return torch.polar(torch.ones_like(ph), ph)


def _to_grid(f):
    """Inverse transform in two dimensions; other lengths than powers of two by
    matrix products, which need no transform plan per length."""
    ny, nx = f.shape
    if nx & (nx - 1) == 0 and ny & (ny - 1) == 0:
        return torch.fft.ifft2(f)
    return (_dft(ny, 1) @ f @ _dft(nx, 1)) / (nx * ny)


def _packet(prob, sigma, p0, center):
    """Normalised positive-energy Gaussian packet, complex128 (2, ny, nx)."""
    x, y, hx, hy = _axes(prob)
    gx = torch.exp(torch.complex(-(x - center[0]) ** 2 / (4 * sigma * sigma), p0[0] * x))
    gy = torch.exp(torch.complex(-(y - center[1]) ** 2 / (4 * sigma * sigma), p0[1] * y))
    # the projector acts on the transform of (g, 0)
    f = (_dft(len(gy), -1) @ gy)[:, None] * (_dft(len(gx), -1) @ gx)[None, :]
    kx = torch.sin(2 * PI * torch.fft.fftfreq(prob["nx"], dtype=torch.float64, device="cuda")) / hx
    ky = torch.sin(2 * PI * torch.fft.fftfreq(prob["ny"], dtype=torch.float64, device="cuda")) / hy
    if prob.get("chirality", 1) < 0:
        ky = -ky
    energy = torch.sqrt(MC2 * MC2 + C_LIGHT ** 2 * (kx[None, :] ** 2 + ky[:, None] ** 2))
    f = f / energy
    psi = torch.empty((2, prob["ny"], prob["nx"]), dtype=torch.complex128, device="cuda")
    psi[0] = _to_grid(0.5 * (energy + MC2) * f)
    psi[1] = _to_grid(0.5 * C_LIGHT * torch.complex(kx[None, :].expand_as(energy), ky[:, None].expand_as(energy)) * f)
    return psi / (math.sqrt(hx * hy) * torch.linalg.vector_norm(psi))


def _momentum(rng, p_max):
    r, v = p_max * math.sqrt(rng.random()), 2 * PI * rng.random()
    return r * math.cos(v), r * math.sin(v)


def _step_inputs(c, seed):
    rng = np.random.default_rng(seed)
    coef = rng.uniform(-c["a0"], c["a0"], size=4 * c["harmonics"]) if c["pulse"] == "fourier" else None
    prob = _problem(c, coef)
    p = _momentum(rng, c["p_max"])
    spread = c["spread"] or 0.1 * min(c["half_x"], c["half_y"])
    center = tuple(rng.uniform(-spread, spread, size=2))
    return prob, _packet(prob, c["sigma"], (p[0] + c["p_x"], p[1]), center)


def _batch_inputs(c, seed):
    """Packets of sizes spread over [n_min, n_max], their states in one buffer."""
    rng = np.random.default_rng(seed)
    # the sizes belong to the case, so that every seed is the same amount of work
    sizes = np.linspace(c["n_min"], c["n_max"], c["packets"]).astype(int)
    probs, psis = [], []
    for n in sizes.tolist():
        half = 0.5 * n * c["h"]
        prob = _problem(_step("", n, n, half, half, c["m"], c["dt"], c["steps"], c["precision"],
                              bz=float(rng.uniform(0.0, 2.0))))
        probs.append(prob)
        psis.append(_packet(prob, 0.2 * half, _momentum(rng, 5.0), tuple(rng.uniform(-0.5 * half, 0.5 * half, size=2))))
    flat = torch.cat([p.reshape(-1) for p in psis])
    views, at = [], 0
    for p in psis:
        views.append(flat[at:at + p.numel()].view(p.shape))
        at += p.numel()
    return probs, flat, views


def _adjoint_inputs(c, seed):
    s = _step("", c["n"], c["n"], c["half"], c["half"], c["m"], c["dt"], c["steps"], "fp64", pulse="fourier",
              harmonics=c["harmonics"], a0=c["a0"], t_pulse=c["t_pulse"], sigma=c["sigma"], p_max=c["p_max"])
    return _step_inputs(s, seed)


def _levels_inputs(c, seed):
    # one point of a scan of the magnetic field about the case's value
    bz = c["bz"] * float(np.random.default_rng([seed, 1]).uniform(0.99, 1.01))
    s = _step("", c["nx"], c["ny"], c["half"], c["half"], 1, 1.0, 1, "fp64", bz=bz, pot_kind=1, pot_z=c["pot_z"],
              pot_a=1.0, sigma=3.0, spread=0.3)
    return _step_inputs(s, seed)


def _hermite_inputs(c, seed):
    rng = np.random.default_rng(seed)
    z = np.exp(np.linspace(math.log(c["z_min"]), math.log(c["z_max"]), c["problems"])) * rng.uniform(0.99, 1.01,
                                                                                                    c["problems"])
    xi, w = np.polynomial.hermite.hermgauss(c["n"])
    sw = np.sqrt(w * np.exp(xi * xi))
    probs, states = [], np.zeros((c["problems"], 2, c["n"], c["n"]), dtype=np.complex128)
    for i, zi in enumerate(z.tolist()):
        probs.append(dict(n=c["n"], scale=1.8 / zi, mass=1.0, c=C_LIGHT, charge=-1.0, bz=c["bz"] * zi * zi, pot_kind=2,
                          pot_z=zi, pot_a=0.0, chirality=int(rng.choice([-1, 1]))))
        gx, gy = (np.exp(-0.5 * (1.8 * xi - o) ** 2) * sw for o in rng.uniform(0.2, 0.5, 2))
        states[i, 0] = np.outer(gy, gx)
        states[i] /= np.linalg.norm(states[i])
    return probs, list(torch.from_numpy(states).cuda())


def prepare(case, seed):
    c = case
    if c["kind"] == "step":
        prob, psi = _step_inputs(c, seed)
        return dict(c=c, psi=psi, prop=binding.Propagator(prob, c["m"], c["precision"], tuning_cache=c["tuned"] or None))
    if c["kind"] == "batch":
        probs, flat, views = _batch_inputs(c, seed)
        return dict(c=c, flat=flat, views=views, prop=binding.BatchPropagator(probs, c["m"], c["precision"]))
    if c["kind"] == "adjoint":
        prob, psi = _adjoint_inputs(c, seed)
        return dict(c=c, psi=psi, prop=binding.Propagator(prob, c["m"], "fp64"))
    if c["kind"] in ("levels", "states"):
        prob, psi = _levels_inputs(c, seed)
        return dict(c=c, psi=psi, prop=binding.Propagator(prob, 1, "fp64", k_eigen=c["k_max"],
                                                          reorth=c["kind"] == "states"))
    probs, states = _hermite_inputs(c, seed)
    lo = [MC2 - 0.6 * p["pot_z"] ** 2 for p in probs]
    hi = [MC2 - 0.4 * p["pot_z"] ** 2 for p in probs]
    return dict(c=c, probs=probs, states=states, lo=lo, hi=hi)


def _filled(values, n):
    """n values, NaN where fewer converged."""
    return np.concatenate([values, np.full(n - len(values), np.nan)])


def run(state):
    """One pass.  Steps return the new state, its norm and the Krylov
    dimensions.  Error estimates and bounds are not among the outputs: they are
    products of many small factors (or residuals at the rounding level) whose
    own last digits say nothing about the result."""
    c = state["c"]
    if c["kind"] == "step":
        st = state["prop"].step(state["psi"], 0.0, c["dt"], c["steps"])
        return {"psi": state["psi"], "norm2": st["norm2"], "k_eff": st["k_eff"]}
    if c["kind"] == "batch":
        st = state["prop"].step(state["views"], 0.0, c["dt"], c["steps"])
        return {"psi": state["flat"], "norm2": np.stack([s["norm2"] for s in st]),
                "k_eff": np.stack([s["k_eff"] for s in st])}
    if c["kind"] == "adjoint":
        loss, grad = state["prop"].adjoint(state["psi"], 0.0, c["dt"], c["steps"], c["every"], c["loss"])
        return {"loss": loss, "grad": grad}
    if c["kind"] == "levels":
        ev, _ = state["prop"].eigen(state["psi"], c["k_max"], MC2 - 2.0, MC2 + c["above"], c["tol"], n_wanted=c["wanted"])
        return {"values": _filled(ev, c["wanted"])}
    if c["kind"] == "states":
        ev, _, vecs = state["prop"].eigen_vectors(state["psi"], c["k_max"], MC2 - 2.0, MC2 + c["above"], c["tol"],
                                                  n_wanted=c["wanted"])
        return {"values": _filled(ev, c["wanted"]), "states": list(vecs)}
    res = binding.hermite_eigen(state["probs"], state["states"], c["k_max"], state["lo"], state["hi"], c["tol"], 1)
    return {"values": np.concatenate([ev for ev, _ in res])}


def work(case):
    """Bytes: each state of the pass read and written once (complex128, two
    components).  Flops: per site and Lanczos iteration one application of H
    (36), the recurrence (16) and its inner products (16), and 16 per vector
    of the recombination (or of a projection and its subtraction)."""
    c = case
    if c["kind"] == "step":
        sites = c["nx"] * c["ny"] * c["steps"]
        return {"bytes": 64 * sites, "flops": sites * c["m"] * 84}
    if c["kind"] == "batch":
        sizes = np.linspace(c["n_min"], c["n_max"], c["packets"]).astype(int)
        sites = int((sizes * sizes).sum()) * c["steps"]
        return {"bytes": 64 * sites, "flops": sites * c["m"] * 84}
    if c["kind"] == "adjoint":
        # a forward and a backward step, and the products of their two bases
        sites = c["n"] * c["n"] * c["steps"]
        return {"bytes": 128 * sites, "flops": sites * (2 * c["m"] * 84 + 16 * c["m"] * c["m"])}
    sites = c.get("nx", 0) * c.get("ny", 0)
    if c["kind"] == "levels":  # the lowest levels converge after about 1000 iterations
        return {"bytes": 32 * sites, "flops": sites * 1000 * 68}
    if c["kind"] == "states":
        k = c["k_max"]
        return {"bytes": 32 * sites * (1 + c["wanted"]), "flops": sites * (k * 68 + k * (k + 1) * 32)}
    return {"bytes": 32 * c["n"] ** 2 * c["problems"], "flops": 16 * c["n"] ** 3 * c["k_max"] * c["problems"]}


# ---------------------------------------------------------------------------
# The same results from plain torch and numpy
# ---------------------------------------------------------------------------
def _field_weights(kind, c, t0, dt):
    """Step averages of the pulse's basis functions by Gauss-Legendre quadrature."""
    u, w = np.polynomial.legendre.leggauss(24)
    t = t0 + 0.5 * dt * (u + 1.0)
    on = np.where((t >= 0) & (t <= c["t_pulse"]), np.sin(PI * t / c["t_pulse"]) ** 2, 0.0)
    if kind == "sin":
        return np.array([0.5 * np.sum(w * on * np.sin(t))])
    out = []
    for k in range(1, c["harmonics"] + 1):
        ph = 2 * PI * k * t / c["t_pulse"]
        out += [0.5 * np.sum(w * on * np.sin(ph)), 0.5 * np.sum(w * on * np.cos(ph))]
    return np.array(out)


def _fields(c, prob, t0, dt):
    """Step-averaged laser vector potential."""
    if c["pulse"] == "none":
        return 0.0, 0.0
    w = _field_weights(c["pulse"], c, t0, dt)
    if c["pulse"] == "sin":
        return 0.0, float(c["a0"] * w[0])
    a = np.asarray(prob["coef"]).reshape(-1, 2, 2)  # harmonic, component, (sin, cos)
    w = w.reshape(-1, 2)
    return float(np.sum(a[:, 0] * w)), float(np.sum(a[:, 1] * w))


class _Lattice:
    """H psi with central differences, and exp(-i dt H) psi, of a problem dict."""

    def __init__(self, prob):
        self.x, self.y, self.hx, self.hy = _axes(prob)
        self.bcx, self.bcy = prob["bc_x"], prob["bc_y"]
        self.chi = -1.0 if prob["chirality"] < 0 else 1.0
        self.ax = (-0.5 * prob["bz"] * self.y)[:, None]
        self.ay = (0.5 * prob["bz"] * self.x)[None, :]
        self.v, vmax = None, 0.0
        if prob["pot_kind"]:
            r2 = self.x[None, :] ** 2 + self.y[:, None] ** 2
            z = prob["pot_z"]
            self.v = -z / torch.sqrt(r2 + prob["pot_a"] ** 2) if prob["pot_kind"] == 1 else -1.5 * z / torch.sqrt(r2 + 3.0 / z ** 2)
            vmax = float(self.v.abs().max())
        self.a_max = (float(self.ax.abs().max()), float(self.ay.abs().max()))
        self.v_max = vmax

    def _diff(self, f, dim, bc, h):
        n = f.shape[dim]
        if bc:
            return (torch.roll(f, -1, dim) - torch.roll(f, 1, dim)) / (2 * h)
        pad = torch.zeros_like(f.narrow(dim, 0, 1))
        g = torch.cat([pad, f, pad], dim)
        return (g.narrow(dim, 2, n) - g.narrow(dim, 0, n)) / (2 * h)

    def apply(self, psi, fx, fy):
        # c sigma1 (p_x + A_x) + c chi sigma2 (p_y + A_y) + mc^2 sigma3 + V (charge -1)
        px = [-1j * self._diff(psi[s], 1, self.bcx, self.hx) + (self.ax + fx) * psi[s] for s in (0, 1)]
        py = [-1j * self._diff(psi[s], 0, self.bcy, self.hy) + (self.ay + fy) * psi[s] for s in (0, 1)]
        up = MC2 * psi[0] + C_LIGHT * (px[1] - 1j * self.chi * py[1])
        dn = -MC2 * psi[1] + C_LIGHT * (px[0] + 1j * self.chi * py[0])
        if self.v is not None:
            up, dn = up + self.v * psi[0], dn + self.v * psi[1]
        return torch.stack([up, dn])

    def exp(self, psi, fx, fy, dt):
        """Chebyshev expansion on [-r, r], r a bound of ||dt H||."""
        hom = sum(abs(float(f.detach() if torch.is_tensor(f) else f)) for f in (fx, fy))
        r = 1.0001 * abs(dt) * (MC2 + self.v_max + C_LIGHT * (1 / self.hx + 1 / self.hy + sum(self.a_max) + hom))
        n = int(r + 12 * r ** (1 / 3) + 24)
        # J_k(r) = (1/N) sum_j cos(k t_j - r sin t_j) over a full period
        t = 2 * PI * np.arange(4 * n) / (4 * n)
        a = [float(np.mean(np.cos(k * t - r * np.sin(t)))) for k in range(n + 1)]
        s = dt / r
        t0, t1 = psi, s * self.apply(psi, fx, fy)
        out = a[0] * t0 + (2 * a[1] * -1j) * t1
        for k in range(2, n + 1):
            t0, t1 = t1, 2 * s * self.apply(t1, fx, fy) - t0
            out = out + (2 * a[k] * (-1j) ** k) * t1
        return out


def _exact_steps(c, prob, psi):
    lat = _Lattice(prob)
    norms = []
    for i in range(c["steps"]):
        psi = lat.exp(psi, *_fields(c, prob, i * c["dt"], c["dt"]), c["dt"])
        norms.append(float(torch.sum(torch.view_as_real(psi) ** 2)))
    return psi, np.array(norms)


def _exact_adjoint(c, seed):
    prob, psi = _adjoint_inputs(c, seed)
    lat = _Lattice(prob)
    coef = torch.tensor(prob["coef"], dtype=torch.float64, requires_grad=True)
    a = coef.reshape(-1, 2, 2)
    psi = psi.clone()
    for i in range(c["steps"]):
        w = torch.from_numpy(_field_weights("fourier", c, i * c["dt"], c["dt"]).reshape(-1, 2))
        f = torch.stack([(a[:, 0] * w).sum(), (a[:, 1] * w).sum()]).cuda()
        psi = checkpoint(lambda p, q: lat.exp(p, q[0], q[1], c["dt"]), psi, f, use_reentrant=False)
    rho = torch.sum(psi.real ** 2 + psi.imag ** 2)
    loss = 0.0
    for bit in range(4):
        if c["loss"] >> bit & 1:
            if bit < 2:
                o = (lat.x[None, None, :] if bit == 0 else lat.y[None, :, None]) * psi
            else:
                o = -1j * torch.stack([lat._diff(psi[s], 3 - bit, (lat.bcx, lat.bcy)[bit - 2], (lat.hx, lat.hy)[bit - 2])
                                       for s in (0, 1)])
            loss = loss + torch.sum((psi.conj() * o).real) / rho
    loss.backward()
    return {"loss": float(loss.detach()), "grad": coef.grad.numpy().copy()}


def _converged(al, be, lo, hi, tol):
    """Clusters of Ritz values of T in the window whose residual is within tol,
    and the eigenvector of each cluster's best member."""
    k = len(al)
    lam, z = np.linalg.eigh(np.diag(al) + np.diag(be[:-1], 1) + np.diag(be[:-1], -1))
    idx = [i for i in range(k) if lo <= lam[i] <= hi]
    out, a = [], 0
    while a < len(idx):
        b = a + 1
        while b < len(idx) and lam[idx[b]] - lam[idx[b - 1]] <= tol:
            b += 1
        members = idx[a:b]
        if be[-1] * np.linalg.norm(z[-1, members]) <= tol:
            best = min(members, key=lambda i: abs(z[-1, i]))
            out.append((float(np.mean(lam[members])), z[:, best] * (-1.0 if z[0, best] < 0 else 1.0)))
        a = b
    return out


def _exact_levels(c, seed):
    """Lanczos on the lattice (with full reorthogonalisation for the states),
    Ritz values every 64 iterations until enough have converged."""
    prob, psi = _levels_inputs(c, seed)
    lat = _Lattice(prob)
    keep = c["kind"] == "states"
    lo, hi = MC2 - 2.0, MC2 + c["above"]
    q = psi / torch.linalg.vector_norm(psi)
    basis = torch.empty((c["k_max"], q.numel()), dtype=torch.complex128, device="cuda") if keep else None
    prev, beta, al, be, found = torch.zeros_like(q), 0.0, [], [], []
    for k in range(1, c["k_max"] + 1):
        z = lat.apply(q, 0.0, 0.0) - beta * prev
        al.append(float(torch.sum((q.conj() * z).real)))
        z = z - al[-1] * q
        if keep:
            basis[k - 1] = q.reshape(-1)
            for _ in range(2):
                z = (z.reshape(-1) - (basis[:k].conj() @ z.reshape(-1)) @ basis[:k]).reshape(q.shape)
        beta = float(torch.linalg.vector_norm(z))
        be.append(beta)
        prev, q = q, z / beta
        if k % 64 == 0 or k == c["k_max"]:
            now = _converged(np.array(al), np.array(be), lo, hi, c["tol"])
            if keep:
                found = now
            else:
                found = sorted(found + [v for v in now if all(abs(v[0] - f[0]) > c["tol"] for f in found)],
                               key=lambda v: v[0])
            if len(found) >= c["wanted"]:
                break
    found = found[:c["wanted"]]
    values = _filled([v for v, _ in found], c["wanted"])
    if not keep:
        return {"values": values}
    vecs = [(torch.from_numpy(t).cuda().to(torch.complex128) @ basis[:len(t)]).reshape(psi.shape) for _, t in found]
    return {"values": values, "states": vecs}


def _exact_hermite(c, seed):
    """The same recurrence for all problems at once, and the lowest Ritz value
    above the window's lower end by bisection on the signs of the pivots."""
    probs, states = _hermite_inputs(c, seed)
    n, b = c["n"], len(probs)
    xi, _ = np.polynomial.hermite.hermgauss(n)
    i = np.arange(n)
    d = np.where(np.eye(n, dtype=bool), 0.0, (-1.0) ** (i[:, None] + i[None, :]) / (xi[:, None] - xi[None, :] + np.eye(n)))
    s = np.array([p["scale"] for p in probs])
    x = s[:, None] * xi[None, :]
    v = np.stack([-1.5 * p["pot_z"] / np.sqrt(xs[None, :] ** 2 + xs[:, None] ** 2 + 3.0 / p["pot_z"] ** 2)
                  for p, xs in zip(probs, x)])
    dm, v, x, bz, chi = (torch.from_numpy(np.asarray(a, dtype=np.float64)).cuda() for a in
                         (d[None] / s[:, None, None], v, x, [p["bz"] for p in probs], [p["chirality"] for p in probs]))
    dt = dm.transpose(1, 2).contiguous()
    ax, ay, chi = -0.5 * bz[:, None, None] * x[:, :, None], 0.5 * bz[:, None, None] * x[:, None, :], chi[:, None, None]

    def mul(a, m, left):
        f = torch.bmm if not left else lambda p, q: torch.bmm(q, p)
        return torch.complex(f(a.real.contiguous(), m), f(a.imag.contiguous(), m))

    def h(q):
        p = [(-1j * mul(q[:, k], dt, False) + ax * q[:, k], -1j * mul(q[:, k], dm, True) + ay * q[:, k]) for k in (0, 1)]
        return torch.stack([(MC2 + v) * q[:, 0] + C_LIGHT * (p[1][0] - 1j * chi * p[1][1]),
                            (v - MC2) * q[:, 1] + C_LIGHT * (p[0][0] + 1j * chi * p[0][1])], 1)

    q = torch.stack(states)
    prev, beta, al, be = torch.zeros_like(q), torch.zeros(b, 1, 1, 1, dtype=torch.float64, device="cuda"), [], []
    for _ in range(c["k_max"]):
        z = h(q) - beta * prev
        a = torch.sum((q.conj() * z).real, (1, 2, 3), keepdim=True)
        z = z - a * q
        beta = torch.sqrt(torch.sum(z.real ** 2 + z.imag ** 2, (1, 2, 3), keepdim=True))
        al.append(a.reshape(b))
        be.append(beta.reshape(b))
        prev, q = q, z / beta
    al, be = torch.stack(al).cpu().numpy(), torch.stack(be).cpu().numpy()

    def lowest(k, n_low=4):
        """The n_low lowest eigenvalues of each T_k above its window's lower end."""
        def count(e):
            t = al[0] - e
            m = (t < 0).astype(int)
            for i in range(1, k):
                t = al[i] - e - be[i - 1] ** 2 / np.where(np.abs(t) < 1e-290, -1e-290, t)
                m += t < 0
            return m

        bottom = MC2 - 0.55 * z2
        below = count(bottom)
        out = []
        for j in range(n_low):
            lo, hi = bottom, MC2 - 0.45 * z2
            for _ in range(60):
                mid = 0.5 * (lo + hi)
                up = count(mid) > below + j
                lo, hi = np.where(up, lo, mid), np.where(up, mid, hi)
            out.append(0.5 * (lo + hi))
        return np.array(out)

    # the ground state (about -z^2/2) and its copies stay where they are as the
    # recurrence goes on; a value on its way to becoming a copy moves
    z2 = np.array([p["pot_z"] for p in probs]) ** 2
    now, before = lowest(c["k_max"]), lowest(c["k_max"] - 64)
    still = np.min(np.abs(now[:, None] - before[None]), 1) <= 1e-7 * (1.0 + 1e-3 * z2)
    return {"values": now[np.argmax(still, 0), np.arange(b)]}


def exact(case, seed):
    c = case
    with torch.set_grad_enabled(c["kind"] == "adjoint"):
        if c["kind"] == "step":
            prob, psi = _step_inputs(c, seed)
            psi, norms = _exact_steps(c, prob, psi)
            return {"psi": psi, "norm2": norms, "k_eff": None}
        if c["kind"] == "batch":
            probs, flat, views = _batch_inputs(c, seed)
            free = dict(pulse="none", **c)
            got = [_exact_steps(free, prob, psi) for prob, psi in zip(probs, views)]
            return {"psi": torch.cat([p.reshape(-1) for p, _ in got]), "norm2": np.stack([v for _, v in got]), "k_eff": None}
        if c["kind"] == "adjoint":
            return _exact_adjoint(c, seed)
        if c["kind"] in ("levels", "states"):
            return _exact_levels(c, seed)
        return _exact_hermite(c, seed)
