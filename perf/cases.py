"""The work that users of this library have it do, as cases that can be timed.

One pass of a case is one request, taken through the public entry points the
way the serving loop does: the initial state is handed over on the device, an
averaging interval is opened, advanced and closed, and every mean is read back
into the caller's device arrays.  Three kinds:

  run       one run (Run): set_state, begin_interval, step, end_interval, read
            (and, where asked for, the strategy-1 remap);
  ensemble  many uneven runs advanced together (Batch.step_static);
  euler     the two-dimensional incompressible test flow (Euler2D).

Grid sizes, precisions, time steps (dt = 0.64 / N), spectra, wave bands and the
ranges of Rossby number and energy ratio are those of the workloads, tests and
benchmarks of this repository.  Intervals are a few to a few tens of steps, so
that a pass is short; everything that happens once per interval is in it.

Mixed-precision runs compute in float32: their means are handed on in float32,
the precision they have.  float64 runs' means stay float64.
"""

import functools
import math

import torch

from paper_2208_02682_amd import OUTPUTS, REMAP_OUTPUTS, Batch, Euler2D, Run, make_config
from paper_2208_02682_amd.autotune import load_default
from paper_2208_02682_amd.lagmean import E2D_OUTPUTS, MOMENTUM_OUTPUTS, field_slots

DEV = "cuda" if torch.cuda.is_available() else "cpu"
SIZES = (64, 128, 192, 256, 384, 512, 1024)
TAU = 2.0 * math.pi


# ------------------------------------------------------------------ the cases

def _run(name, n, precision, steps, **kw):
    c = {"name": name, "kind": "run", "n": n, "precision": precision, "steps": steps, "k0": 6.0 * n / 64, "ro": 0.05,
         "ratio": 1.0, "interp": "bilinear", "fields": "h,zeta", "momentum": False, "remap": False}
    c.update(kw)
    return c


def listed():
    return [
        # the smallest configuration, float64: launches and latency count
        _run("run 64 fp64", 64, "fp64", 31),
        # the most frequent request of the serving mix
        _run("run 128 fp32", 128, "fp32", 40),
        # a grid that is not a power of two
        _run("run 192 fp32", 192, "fp32", 33),
        # the 256 x 256 float64 workload, with strategy 1 remapped to mean positions
        _run("run 256 fp64 remap", 256, "fp64", 30, k0=12.0 / math.sqrt(2.0), remap=True),
        # every option of strategy 2 at once: cubic gathers, the momentum 1-form,
        # and the velocity and potential vorticity as averaged fields
        _run("run 384 fp32 cubic", 384, "fp32", 24, interp="cubic", fields="u,q", momentum=True),
        # the large request of the serving mix
        _run("run 512 fp32", 512, "fp32", 40),
        # the headline workload: 1024 x 1024, mixed precision
        _run("run 1024 fp32", 1024, "fp32", 48, k0=32.0 / math.sqrt(2.0), ro=0.1),
        # the same grid entirely in float64
        _run("run 1024 fp64", 1024, "fp64", 10, k0=32.0 / math.sqrt(2.0), ro=0.1),
        # an ensemble of the smallest configuration
        {"name": "ensemble 64 fp64", "kind": "ensemble", "count": 32, "n_lo": 64, "n_hi": 64, "precision": "fp64",
         "steps_lo": 12, "steps_hi": 20},
        # uneven mixed-precision runs, as the batched workload has them
        {"name": "ensemble uneven fp32", "kind": "ensemble", "count": 24, "n_lo": 128, "n_hi": 512, "precision": "fp32",
         "steps_lo": 9, "steps_hi": 16},
        # the two-vortex test at its own size
        {"name": "euler 128 bilinear", "kind": "euler", "n": 128, "steps": 50, "interp": "bilinear"},
        # and on a large grid with cubic gathers
        {"name": "euler 512 cubic", "kind": "euler", "n": 512, "steps": 15, "interp": "cubic"},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["run", "run", "run", "ensemble", "euler"])
    if kind == "ensemble":
        lo, hi = sorted(rng.choice(SIZES[:6]) for _ in range(2))
        count = _log_int(rng, 3, 24 if hi <= 256 else 12)
        return {"kind": kind, "count": count, "n_lo": lo, "n_hi": hi, "precision": rng.choice(["fp32", "fp64", "both"]),
                "steps_lo": rng.randint(3, 6), "steps_hi": rng.randint(7, 14)}
    if kind == "euler":
        n = rng.choice(SIZES)
        return {"kind": kind, "n": n, "steps": _log_int(rng, 3, max(4, min(40, 1 << 22 >> (2 * n.bit_length() - 2)))),
                "interp": rng.choice(["bilinear", "cubic"])}
    n = rng.choice(SIZES)
    precision = rng.choice(["fp32", "fp64"])
    plain = rng.random() < 0.6  # the default options
    most = (40 if precision == "fp32" else 25) if n < 1024 else (24 if precision == "fp32" else 7)
    c = _run("", n, precision, _log_int(rng, 3, most if plain else max(4, most // 2)),
             k0=rng.uniform(1.4, 6.0) * n / 64, ro=rng.uniform(0.02, 0.2),
             ratio=math.exp(rng.uniform(math.log(0.25), math.log(4.0))))
    del c["name"]
    if not plain:
        c["interp"] = rng.choice(["bilinear", "cubic"])
        c["fields"] = rng.choice(["h,zeta", "h,u", "zeta,v", "u,v", "u,q", "h,q"])
        c["momentum"] = rng.random() < 0.5
    c["remap"] = rng.random() < 0.25
    return c


def _members(case, seed):
    """The runs of an ensemble: grid sizes spread evenly over the case's range, uneven interval lengths."""
    sizes = [n for n in SIZES if case["n_lo"] <= n <= case["n_hi"]]
    out = []
    for i in range(case["count"]):
        n = sizes[i % len(sizes)]
        p = case["precision"] if case["precision"] != "both" else ("fp32", "fp32", "fp64")[i % 3]
        steps = case["steps_lo"] + (7 * i) % (case["steps_hi"] - case["steps_lo"] + 1)
        f = (i + 0.5) / case["count"]
        out.append((_run("", n, p, steps, ro=0.02 + 0.18 * f, ratio=0.25 * 16.0 ** ((0.37 + 5 * f) % 1.0)),
                    seed * 1000 + i))
    return out


# ----------------------------------------------------------- the initial states

@functools.lru_cache(maxsize=16)
def _wavenumbers(n):
    k = torch.fft.fftfreq(n, d=1.0 / n, dtype=torch.float64).to(DEV)
    return k[None, :].expand(n, n), k[:, None].expand(n, n)


def _flow(c, seed):
    """Turbulence in geostrophic balance plus a band of Poincare waves (f = g = H = 1):
    geostrophic shell spectrum k^4 exp(-(k / k0)^2) with rms speed ro, waves in
    [k0 / 3, 2 k0 / 3] with the given wave / vortex energy ratio, random phases."""
    n, k0 = c["n"], c["k0"]
    kx, ky = _wavenumbers(n)
    k2 = kx * kx + ky * ky
    kk = k2.sqrt()
    g = torch.Generator().manual_seed(seed)
    ph = (TAU * torch.rand(2, n, n, generator=g, dtype=torch.float64)).to(DEV)
    cut = (n - 1) // 3
    inside = (kx.abs() <= cut) & (ky.abs() <= cut) & (kk > 0)

    def real(a):
        return torch.fft.ifft2(a).real * (n * n)

    psi = torch.polar(torch.where(inside, kk.sqrt() * torch.exp(-k2 / (2 * k0 * k0)), torch.zeros_like(kk)), ph[0])
    ug, vg, eg = real(-1j * ky * psi), real(1j * kx * psi), real(psi)
    s = c["ro"] / (ug * ug + vg * vg).mean().sqrt()
    ug, vg, eg = ug * s, vg * s, eg * s
    band = (kk >= k0 / 3) & (kk <= 2 * k0 / 3) & (kk > 0)
    w = torch.polar(band.double(), ph[1])
    om, safe = (1 + k2).sqrt(), torch.where(band, k2, torch.ones_like(k2))
    uw, vw, ew = real(w * (om * kx + 1j * ky) / safe), real(w * (om * ky - 1j * kx) / safe), real(w)
    a = (c["ratio"] * (ug * ug + vg * vg + eg * eg).mean() / (uw * uw + vw * vw + ew * ew).mean()).sqrt()
    return (ug + a * uw).contiguous(), (vg + a * vw).contiguous(), (1.0 + eg + a * ew).contiguous()


def _vorticity(n, seed):
    """Two like-signed Gaussian vortices near their places in the paper's test (moved a little by the seed)."""
    g = torch.Generator().manual_seed(seed)
    d = (0.2 * torch.rand(4, generator=g, dtype=torch.float64) - 0.1).tolist()
    x = torch.arange(n, dtype=torch.float64, device=DEV) * (TAU / n)
    X, Y, pi = x[None, :], x[:, None], math.pi
    return (torch.exp(-(X - pi + 0.1 + d[0]) ** 2 - (Y - pi + pi / 3 + d[1]) ** 2)
            + torch.exp(-(X - pi - 0.1 + d[2]) ** 2 - (Y - pi - pi / 3 + d[3]) ** 2)).contiguous()


def _dt(n):
    return 0.64 / n


def _nu8(n):
    return 0.1 / (_dt(n) * float((n - 1) // 3) ** 8)


# ------------------------------------------------------------------- the passes

@functools.lru_cache(maxsize=1)
def _schedules():
    return load_default("gfx950")  # the shipped launch schedules, once per process


def _config(c):
    return make_config(c["n"], precision=c["precision"], dt=_dt(c["n"]), nu8=_nu8(c["n"]), interp=c["interp"],
                       momentum=c["momentum"], fields=tuple(c["fields"].split(",")))


def _reads(c, cfg):
    """name -> (field, kind) of every output of a run, the means named by the averaged fields."""
    slots = field_slots(cfg)
    out = {}
    for name, fk in OUTPUTS.items():
        out[f"{name.split(':')[0]}:{slots[fk[0]]}" if ":" in name else name] = fk
    if c["momentum"]:
        out.update(MOMENTUM_OUTPUTS)
    if c["remap"]:
        for name, fk in REMAP_OUTPUTS.items():
            out[f"{name.split(':')[0]}:{slots[fk[0]]}" if ":" in name else name] = fk
    return out


def prepare(case, seed):
    _schedules()
    stream = torch.cuda.current_stream().cuda_stream
    if case["kind"] == "euler":
        n = case["n"]
        flow = Euler2D(n, _dt(n), interp=case["interp"], stream=stream)
        return {"kind": "euler", "flow": flow, "steps": case["steps"], "zeta": _vorticity(n, seed),
                "out": {k: torch.empty(n, n, dtype=torch.float64, device=DEV) for k in E2D_OUTPUTS}}
    if case["kind"] == "run":
        cfg = _config(case)
        reads = _reads(case, cfg)
        out = torch.empty(len(reads), case["n"], case["n"], dtype=torch.float64, device=DEV)
        return {"kind": "run", "run": Run(cfg, stream=stream), "state": _flow(case, seed), "steps": case["steps"],
                "remap": case["remap"], "reads": reads, "out": out, "fp32": case["precision"] == "fp32"}
    members, total = [], {}
    for c, s in _members(case, seed):
        at = total.get(c["precision"], 0)
        total[c["precision"]] = at + c["n"] ** 2
        members.append({"run": Run(_config(c), stream=stream), "state": _flow(c, s), "steps": c["steps"], "n": c["n"],
                        "precision": c["precision"], "at": at})
    out = {p: torch.empty(len(OUTPUTS), t, dtype=torch.float64, device=DEV) for p, t in total.items()}
    return {"kind": "ensemble", "batch": Batch(stream=stream), "members": members, "out": out}


def run(state):
    if state["kind"] == "euler":
        e = state["flow"]
        e.set_vorticity(state["zeta"])
        e.begin_interval()
        e.step(state["steps"])
        e.end_interval()
        return {k: e.read(k, out=o) for k, o in state["out"].items()}
    if state["kind"] == "run":
        r, out = state["run"], state["out"]
        r.set_state(*state["state"])
        r.begin_interval()
        r.step(state["steps"])
        r.end_interval()
        if state["remap"]:
            r.remap_s1()
        for i, (field, kind) in enumerate(state["reads"].values()):
            r.read_mean(field, kind, out=out[i])
        if state["fp32"]:
            out = out.float()
        return {name: out[i] for i, name in enumerate(state["reads"])}
    batch = state["batch"]
    for m in state["members"]:
        m["run"].set_state(*m["state"])
        m["run"].begin_interval()
        batch.add(m["run"], m["steps"])
    while batch.step_static(32):
        pass
    for m in state["members"]:
        r, n = m["run"], m["n"]
        batch.remove(r)
        r.end_interval()
        for i, (field, kind) in enumerate(OUTPUTS.values()):
            r.read_mean(field, kind, out=state["out"][m["precision"]][i, m["at"]:m["at"] + n * n].view(n, n))
    outs = {p: o.float() if p == "fp32" else o for p, o in state["out"].items()}
    return {f"{p} {name}": o[i] for p, o in outs.items() for i, name in enumerate(OUTPUTS)}


# ---------------------------------------------------- what a pass cannot do without

def _transform_flops(n):
    return 2.5 * n * n * math.log2(n * n)  # one real two-dimensional transform


def _run_work(c):
    """State read and written once a step (2/3-rule modes only; xi and P in float64),
    initial fields in and means out; the transforms and products of four stages."""
    n, k = c["n"], (c["n"] - 1) // 3
    size = 8 if c["precision"] == "fp32" else 16
    modes = (k + 1) * (2 * k + 1)
    fields = 9 + (2 if c["momentum"] else 0)
    state = modes * (fields * size * (2 if c["precision"] == "fp32" else 1) + 4 * 16)
    outs = 10 + (2 if c["momentum"] else 0) + (4 if c["remap"] else 0)
    inverse, forward = (22 + 8, 15) if c["momentum"] else (22, 13)
    points = 150 if c["interp"] == "bilinear" else 300
    return {"bytes": c["steps"] * 2 * state + (3 + outs) * n * n * 8,
            "flops": c["steps"] * 4 * ((inverse + forward) * _transform_flops(n) + points * n * n)}


def work(case):
    if case["kind"] == "run":
        return _run_work(case)
    if case["kind"] == "ensemble":
        each = [_run_work(c) for c, _ in _members(case, 0)]
        return {k: sum(w[k] for w in each) for k in ("bytes", "flops")}
    n, k = case["n"], (case["n"] - 1) // 3
    state = (k + 1) * (2 * k + 1) * 4 * 16 + 4 * n * n * 8  # spectral fields, and semi-Lagrangian ones on the grid
    return {"bytes": case["steps"] * 2 * state + 8 * n * n * 8,
            "flops": case["steps"] * ((2 * (11 + 4) + 3) * _transform_flops(n) + (200 if case["interp"] == "cubic" else 100) * n * n)}


# --------------------------------------------------- the same numbers in 64 bits

class _Grid:
    def __init__(self, n):
        self.n, self.dx = n, TAU / n
        k = torch.fft.fftfreq(n, d=1.0 / n, dtype=torch.float64).to(DEV)
        self.kx = torch.arange(n // 2 + 1, dtype=torch.float64, device=DEV)[None, :]
        self.ky = k[:, None]
        cut = (n - 1) // 3
        self.mask = ((self.kx <= cut) & (self.ky.abs() <= cut)).double()
        self.j = torch.arange(n, device=DEV)

    def to(self, a):
        return self.mask * torch.fft.rfft2(a)

    def back(self, a):
        return torch.fft.irfft2(a, s=(self.n, self.n))

    def dx_(self, a):
        return self.back(1j * self.kx * a)

    def dy_(self, a):
        return self.back(1j * self.ky * a)

    def at(self, f, ox, oy, cubic):
        """Periodic bilinear or 4 x 4-point Lagrange interpolants of the fields f at every grid point plus (ox, oy)."""
        px, py = ox / self.dx, oy / self.dx
        fx, fy = px.floor(), py.floor()

        def weights(a):
            if not cubic:
                return {0: 1 - a, 1: a}
            return {-1: -a * (a - 1) * (a - 2) / 6, 0: (a + 1) * (a - 1) * (a - 2) / 2, 1: -(a + 1) * a * (a - 2) / 2,
                    2: (a + 1) * a * (a - 1) / 6}

        ix, iy = self.j[None, :] + fx.long(), self.j[:, None] + fy.long()
        out = torch.zeros_like(f)
        for b, wy in weights(py - fy).items():
            for a, wx in weights(px - fx).items():
                out += (wx * wy) * f[..., (iy + b) % self.n, (ix + a) % self.n]
        return out


def _exact_run(c, seed):
    n, dt, nu8 = c["n"], _dt(c["n"]), _nu8(c["n"])
    G, cubic = _Grid(n), c["interp"] == "cubic"
    names = sorted(c["fields"].split(","), key=["h", "zeta", "u", "v", "q"].index)
    k8 = nu8 * (G.kx ** 2 + G.ky ** 2) ** 4
    # u, v, h | xi | g-bar | g-tilde | P | Eulerian | momentum
    Y = torch.zeros(15 if c["momentum"] else 13, n, n // 2 + 1, dtype=torch.complex128, device=DEV)
    Y[:3] = G.to(torch.stack(_flow(c, seed)))

    def rhs(Y, s):
        p = G.back(Y)
        u, v, h = p[0], p[1], p[2]
        z = G.back(1j * (G.kx * Y[1] - G.ky * Y[0]))
        R = torch.empty_like(Y)
        B = Y[2] + G.to(0.5 * (u * u + v * v))
        R[0] = G.to(z * v) + Y[1] - 1j * G.kx * B - k8 * Y[0]
        R[1] = -G.to(z * u) - Y[0] - 1j * G.ky * B - k8 * Y[1]
        R[2] = -1j * G.kx * G.to(h * u) - 1j * G.ky * G.to(h * v) - k8 * Y[2]
        f = torch.stack([{"h": h - 1.0, "zeta": z, "u": u, "v": v, "q": (1.0 + z) / h}[m] for m in names])
        xi = p[3:5]
        w = xi / s if s > 0 else 0.5 * p[0:2]
        at = G.at(torch.cat([p[0:2], f]), xi[0], xi[1], cubic)
        dx, dy = G.dx_(Y[3:]), G.dy_(Y[3:])
        R[3:5] = G.to(at[:2] - w - (w[0] * dx[0:2] + w[1] * dy[0:2]))
        R[5:7] = G.to(at[2:] - (w[0] * dx[2:4] + w[1] * dy[2:4]))
        R[7:9] = G.to(f - (u * dx[4:6] + v * dy[4:6]))
        R[9:11] = G.to(s * p[0:2] - (u * dx[6:8] + v * dy[6:8]))
        R[11:13] = G.to(f)
        if c["momentum"]:
            g = p[13:15]
            for i, d in enumerate((dx, dy)):
                e = torch.zeros(2, 1, 1, dtype=torch.float64, device=DEV)
                e[i] = 1.0
                r = (at[:2] * (e + d[0:2])).sum(0) - (w[0] * dx[10 + i] + w[1] * dy[10 + i])
                if s > 0:
                    r = r - (g * d[0:2]).sum(0) / s
                R[13 + i] = G.to(r)
        return R

    for m in range(c["steps"]):
        k1 = rhs(Y, m * dt)
        k2 = rhs(Y + 0.5 * dt * k1, (m + 0.5) * dt)
        k3 = rhs(Y + 0.5 * dt * k2, (m + 0.5) * dt)
        k4 = rhs(Y + dt * k3, (m + 1.0) * dt)
        Y = Y + dt / 6.0 * (k1 + 2 * k2 + 2 * k3 + k4)
    T = c["steps"] * dt
    p = G.back(Y)
    off = torch.tensor([1.0 if m == "h" else 0.0 for m in names], dtype=torch.float64, device=DEV)[:, None, None]
    s2, s1, eu, eta = p[5:7] / T + off, p[7:9] / T + off, p[11:13] / T + off, p[9:11] / T
    out = {"S2_xi_x": p[3], "S2_xi_y": p[4], "S1_eta_x": eta[0], "S1_eta_y": eta[1]}
    for i, m in enumerate(names):
        out.update({f"S2_mean:{m}": s2[i], f"S1_mean:{m}": s1[i], f"E_mean:{m}": eu[i]})
    if c["momentum"]:
        out.update({"S2_mom_x": p[13] / T, "S2_mom_y": p[14] / T})
    if c["remap"]:
        # the end position x of the particle with mean position y solves x - eta(x) = y (eta is a contraction here)
        d = torch.zeros_like(eta)
        for _ in range(200):
            last, d = d, G.at(eta, d[0], d[1], False)
            if float((d - last).abs().max()) < 1e-15:
                break
        means = G.at(s1, d[0], d[1], False)
        out.update({f"S1R_mean:{m}": means[i] for i, m in enumerate(names)})
        out.update({"S1R_xi_x": d[0], "S1R_xi_y": d[1]})
    return out


def _exact_euler(c, seed):
    n, dt, cubic = c["n"], _dt(c["n"]), c["interp"] == "cubic"
    G = _Grid(n)
    k2 = G.kx ** 2 + G.ky ** 2
    inv = torch.where(k2 > 0, 1.0 / k2, torch.zeros_like(k2))
    Y = torch.zeros(4, n, n // 2 + 1, dtype=torch.complex128, device=DEV)  # zeta, g-tilde, P
    Y[0] = G.to(_vorticity(n, seed))

    def velocity(z):
        return G.back(torch.stack([1j * G.ky * inv * z, -1j * G.kx * inv * z]))

    def rhs(Y, s):
        u, v = vel = velocity(Y[0])
        src = torch.cat([torch.zeros_like(vel[:1]), G.back(Y[:1]), s * vel])
        return G.to(src - (u * G.dx_(Y) + v * G.dy_(Y)))

    sl = torch.zeros(4, n, n, dtype=torch.float64, device=DEV)  # f~, eta, and zeta at the last step
    sl[3] = G.back(Y[0])
    for m in range(c["steps"]):
        k1 = rhs(Y, m * dt)
        Y = Y + 0.5 * dt * (k1 + rhs(Y + dt * k1, (m + 1) * dt))
        d, z = dt * velocity(Y[0]), G.back(Y[0])
        a = G.at(sl, -d[0], -d[1], cubic)
        sl = torch.cat([((m * a[0] + 0.5 * (a[3] + z)) / (m + 1))[None], (m * a[1:3] + (m + 0.5) * d) / (m + 1), z[None]])
    T, p = c["steps"] * dt, G.back(Y)
    return {"zeta": p[0], "PS_mean": p[1] / T, "PS_eta_x": p[2] / T, "PS_eta_y": p[3] / T, "SL_mean": sl[0],
            "SL_eta_x": sl[1], "SL_eta_y": sl[2]}


def exact(case, seed):
    if case["kind"] == "run":
        return _exact_run(case, seed)
    if case["kind"] == "euler":
        return _exact_euler(case, seed)
    parts = {}
    for c, s in _members(case, seed):
        for name, a in _exact_run(c, s).items():
            parts.setdefault(f"{c['precision']} {name}", []).append(a.reshape(-1))
    return {k: torch.cat(v) for k, v in parts.items()}
