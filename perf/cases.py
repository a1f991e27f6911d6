"""Timed cases of the M2M step: what a user of this package has it do.

A case is one call pattern at one size:

* ``fit``:     a fit that is already set up takes ``steps`` M2M steps (``Fit.step``);
               with ``monitor`` the program then reads the observables and chi^2,
               as a loop that watches its convergence does;
* ``batch``:   a set of fits that step together takes ``steps`` steps (``Batch.run``);
* ``observe``: a particle realization is measured (``Fit.observe``), the call that
               builds targets.

The particle models, targets and 64-bit reference values are made here with
plain torch and numpy; the package is used only for what is timed.
"""

from __future__ import annotations

import math

import numpy as np
import torch

from paper_1202_2355_amd import tuning
from paper_1202_2355_amd.batch import Batch
from paper_1202_2355_amd.fit import Fit

F64 = torch.float64
FIELDS = ("x", "y", "z", "vx", "vy", "vz")
GRID = {"v2": (20, 10), "none": (20, 10), "gh": (50, 20), "losvd": (64, 32)}
# more than this does not fit the registers and LDS of the chip together, so
# that every step has to stream it
ON_CHIP = 128 << 20


# ------------------------------------------------------------------ the cases
def _case(name=None, kind="fit", kin="gh", dtype="f32", n=1_000_000, steps=50, **kw):
    c = {"kind": kind, "kin": kin, "dtype": dtype, "n": n, "steps": steps,
         "fits": 1, "n_hi": 0, "monitor": False, "nfw": False, "halo": False, "alm": -1, "scf": -1,
         "smooth": False, "gh": 4, "entropy": "mpr"}
    c.update(kw)
    if name is not None:
        c["name"] = name
    return c


def listed():
    return [
        # the smallest call: one step of a fit of a few thousand particles, as an
        # interactive session or a smoke test makes it
        _case("step_gh_4k", n=4001, steps=1),
        # a whole small fit in FP64 state (200 steps, 2e4 particles), its observables read at the end
        _case("fit_v2_f64_20k", kin="v2", dtype="f64", n=20_000, steps=200, monitor=True),
        # the paper's scale: 1e6 particles, Gauss-Hermite data, FP32 state
        _case("fit_gh_1m", n=1_000_000, steps=100),
        # FP64 state of an ordinary odd size (reference runs, convergence checks)
        _case("fit_gh_f64_300k", dtype="f64", n=300_007, steps=30),
        # the largest single fit: 8e6 particles in a Hernquist + NFW potential, LOSVD data
        _case("fit_losvd_8m", kin="losvd", n=8_000_000, steps=30, nfw=True),
        # the batched default workload: 64 fits of 2^16..2^21 particles, 3.6e7 in all
        _case("batch64_gh", kind="batch", n=1 << 16, n_hi=1 << 21, fits=64, steps=26, nfw=True),
        # a server's turn of 64 steps over 16 requests of 1e5..1e6 particles
        _case("batch16_losvd", kind="batch", kin="losvd", n=100_000, n_hi=1_000_000, fits=16, steps=64,
              nfw=True),
        # a scan over the mass-to-light ratio of a rotating model in a
        # logarithmic halo: a few small fits, prior cells split by the sense of rotation
        _case("scan8_v2_f64_halo", kind="batch", kin="v2", dtype="f64", n=30_011, n_hi=30_011, fits=8,
              steps=64, halo=True),
        # targets: a 2^22-particle realization measured as line-of-sight histograms
        _case("observe_losvd_4m", kind="observe", kin="losvd", n=1 << 22, steps=1, nfw=True),
        # spherical-harmonic density observables (l <= 4 on a 60-point mesh)
        _case("fit_alm4_1m", n=1_000_000, steps=26, alm=4),
        # the stellar potential from the particles (l <= 4, rebuilt every 10 steps)
        _case("fit_scf4_1m", n=1_000_000, steps=26, scf=4),
        # thin-plate smoothing of the prior grid at every refresh
        _case("fit_smooth_gh_200k", n=200_003, steps=52, smooth=True),
    ]


def draw(rng):
    """One more case of the same ranges: sizes spread over their logarithm,
    odd ones among them."""
    def size(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    what = rng.choice(("step", "fit", "fit", "fit", "batch", "batch", "observe", "option", "option"))
    kin = rng.choice(("v2", "gh", "gh", "losvd", "losvd"))
    dtype = rng.choice(("f32", "f32", "f64"))
    nfw = rng.random() < 0.5
    gh = rng.choice((4, 4, 2, 6))
    if what == "step":
        return _case(kin=kin, dtype=dtype, gh=gh, n=size(1000, 300_000), steps=rng.randint(1, 4), nfw=nfw,
                     monitor=dtype == "f64")
    if what == "fit":
        return _case(kin=kin, dtype=dtype, gh=gh, n=size(5000, 4_000_000 if dtype == "f32" else 1_000_000),
                     steps=rng.randint(26, 60), nfw=nfw, monitor=dtype == "f64",
                     entropy=rng.choice(("mpr", "mpr", "mpr", "gwr")))
    if what == "batch":
        lo = size(10_000, 200_000)
        return _case(kind="batch", kin=kin, dtype=dtype, n=lo, n_hi=lo * rng.randint(1, 6),
                     fits=rng.randint(3, 12), steps=rng.randint(26, 64), nfw=nfw, halo=rng.random() < 0.3)
    if what == "observe":
        return _case(kind="observe", kin=kin, dtype=dtype, n=size(20_000, 4_000_000), steps=1, nfw=nfw)
    opt = rng.choice(("alm", "scf", "smooth"))
    n, steps = size(10_000, 800_000), rng.randint(11, 27)
    if opt == "alm":
        return _case(kin=kin, dtype=dtype, n=n, steps=steps, alm=rng.choice((2, 3, 4)))
    if opt == "scf":
        return _case(kin=kin, dtype=dtype, n=n, steps=steps, scf=rng.choice((2, 3, 4)), nfw=nfw)
    return _case(kin=kin, dtype=dtype, n=n, steps=rng.randint(26, 52), smooth=True, nfw=nfw)


# ------------------------------------------------------- potential and layout
def _potential(case, k=0, count=1):
    """Potential k of `count`: mass-to-light ratios 0.5..2 over a batch, an
    NFW halo of concentration 5..15, or the logarithmic halo."""
    f = (k + 0.5) / count
    p = dict(G=1.0, M_star=1.0, a=1.0, upsilon=1.0 if count == 1 else 0.5 + 1.5 * f, M200=0.0, c=0.0,
             r_s=0.0, v0=0.0, r0=1.0, q=1.0)
    if case["nfw"]:
        p.update(M200=10.0, c=8.0 if count == 1 else 5.0 + 10.0 * ((k * 0.618) % 1.0))
        p["r_s"] = 100.0 / p["c"]
    if case["halo"]:
        p.update(v0=0.4, r0=5.0, q=0.8)
    return p


def _layout(case):
    kin = case["kin"]
    n_r, n_R = {"v2": (30, 20), "gh": (40, 30), "losvd": (50, 40)}[kin]
    lay = dict(n_r=n_r, r_min=0.05, r_max=20.0, n_R=n_R, R_min=0.05, R_max=20.0, kin=kin, gh_nmax=0,
               n_v=0, v_min=0.0, v_max=0.0, dens="bins", l_max=0)
    if kin == "gh":
        lay["gh_nmax"] = case["gh"]
    if kin == "losvd":
        lay.update(n_v=64, v_min=-4.0, v_max=4.0)
    if case["alm"] >= 0:
        lay.update(n_r=60, dens="alm", l_max=case["alm"])
    return lay


def _params(case, pot):
    n_E, n_x = GRID[case["kin"]]
    P = _Pot(pot)
    lo = float(P.phi(torch.zeros(1, dtype=F64)))
    hi = float(P.phi(torch.full((1,), 20.0, dtype=F64))) if case["halo"] else 0.0
    par = dict(dt=0.01, eps=0.1, mu=1e-2, alpha=2.1, mass=1.0, entropy=case["entropy"], n_E=n_E, n_x=n_x,
               prior_every=25, E_lo=lo, E_hi=hi, smooth=int(case["smooth"]), cells=3 if case["halo"] else 0)
    if case["scf"] >= 0:
        par.update(scf_lmax=case["scf"], scf_nr=32, scf_rmin=0.02, scf_rmax=100.0, scf_every=10)
    return par


class _Pot:
    """Hernquist stars, an NFW halo and a flattened logarithmic halo in 64 bits."""

    def __init__(self, p):
        self.gm, self.a = p["G"] * p["M_star"] * p["upsilon"], p["a"]
        self.gn = p["G"] * p["M200"] / (math.log1p(p["c"]) - p["c"] / (1 + p["c"])) if p["M200"] > 0 else 0.0
        self.rs = p["r_s"] if p["M200"] > 0 else 1.0
        self.v2, self.r02, self.iq2 = p["v0"] ** 2, p["r0"] ** 2, 1.0 / p["q"] ** 2

    def phi(self, r):
        """At radius r in the equatorial plane."""
        v = -self.gm / (r + self.a)
        if self.gn:
            v = v - self.gn * torch.where(r > 0, torch.log1p(r / self.rs) / r.clamp_min(1e-300), 1.0 / self.rs)
        if self.v2:
            v = v + 0.5 * self.v2 * torch.log(self.r02 + r * r)
        return v

    def mass(self, r, stars=True):
        """G M(<r) of the spherical parts."""
        m = self.gm * r * r / (r + self.a) ** 2 if stars else torch.zeros_like(r)
        if self.gn:
            q = r / self.rs
            m = m + self.gn * (torch.log1p(q) - q / (1 + q))
        return m

    def vc2(self, r):
        v = self.mass(r) / r
        return v + self.v2 * r * r / (self.r02 + r * r) if self.v2 else v

    def accel(self, x, y, z, stars=True):
        r = torch.sqrt(x * x + y * y + z * z)
        s = self.mass(r, stars) / r ** 3
        sz = s
        if self.v2:
            h = self.v2 / (self.r02 + x * x + y * y + z * z * self.iq2)
            s, sz = s + h, s + h * self.iq2
        return -s * x, -s * y, -sz * z


# ----------------------------------------------------------- particle models
def _model(case, pot, n, g, anisotropic=False):
    """n particles in 64 bits: a Hernquist (Plummer for LOSVD data) tracer with
    Gaussian velocities of the Jeans dispersion, redrawn until bound; the
    target realizations are radially anisotropic beyond r = 1."""
    P, dev = _Pot(pot), "cuda"
    u = torch.rand(n, generator=g, device=dev, dtype=F64).clamp_(1e-12, 1 - 1e-9)
    plummer = case["kin"] == "losvd"
    r = 1.0 / torch.sqrt(u.pow(-2.0 / 3.0) - 1.0) if plummer else torch.sqrt(u) / (1 - torch.sqrt(u))
    rt = torch.logspace(-7, 6, 2000, dtype=F64)
    rho = (1 + rt * rt) ** -2.5 if plummer else 1 / (rt * (1 + rt) ** 3)
    f = rho * P.vc2(rt)  # rho dPhi/dr dr = rho v_c^2 dln r
    d = 0.5 * (f[1:] + f[:-1]) * math.log(10.0) * 13 / 1999
    s2 = (torch.cat([d.flip(0).cumsum(0).flip(0), torch.zeros(1, dtype=F64)]) / rho).to(dev)
    pos = ((torch.log10(r) + 7) * (1999 / 13)).clamp(0, 1998.999)
    i = pos.long()
    sig = torch.sqrt((s2[i] + (pos - i) * (s2[i + 1] - s2[i])).clamp_min(1e-12))
    psi = P.phi(torch.tensor([1e4], dtype=F64, device=dev)) - P.phi(r) if case["halo"] else -P.phi(r)
    psi = psi.clamp_min(1e-12)
    v = torch.randn(3, n, generator=g, device=dev, dtype=F64) * sig
    for _ in range(6):
        bad = 0.5 * (v * v).sum(0) >= psi
        v = torch.where(bad, torch.randn(3, n, generator=g, device=dev, dtype=F64) * sig * 0.7, v)
    v = torch.where(0.5 * (v * v).sum(0) >= psi, 0.1 * v, v)
    if anisotropic:
        v[1:] /= torch.sqrt(1 + r * r)
    ct = 2 * torch.rand(n, generator=g, device=dev, dtype=F64) - 1
    ph = 2 * math.pi * torch.rand(n, generator=g, device=dev, dtype=F64)
    st, cp, sp = torch.sqrt((1 - ct * ct).clamp_min(0)), torch.cos(ph), torch.sin(ph)
    out = (r * st * cp, r * st * sp, r * ct,
           v[0] * st * cp + v[1] * ct * cp - v[2] * sp, v[0] * st * sp + v[1] * ct * sp + v[2] * cp,
           v[0] * ct - v[1] * st)
    return dict(zip(FIELDS, out))


def _rounded(p, dtype):
    t = torch.float64 if dtype == "f64" else torch.float32
    return {k: v.to(t) for k, v in p.items()}


# -------------------------------------------------------- observables, 64 bits
def _log_edges(lo, hi, n):
    e = lo * (hi / lo) ** (np.arange(n + 1) / n)
    e[0], e[-1] = lo, hi
    return torch.tensor(e, dtype=F64, device="cuda")


def _bin(v, e):
    k = torch.bucketize(v, e, right=True) - 1
    return torch.where((v >= e[0]) & (v < e[-1]), k, -1)


def _direction(x, y, z):
    R = torch.sqrt(x * x + y * y)
    r = torch.sqrt(R * R + z * z)
    return z / r, R / r, x / R, y / R


def _harmonics(L, ct, st, cp, sp):
    """(l^2 + l + m, Y_lm): real orthonormal harmonics, Condon-Shortley phase."""
    pmm, cm, sm = torch.full_like(ct, 0.5 / math.sqrt(math.pi)), torch.ones_like(ct), torch.zeros_like(ct)
    for m in range(L + 1):
        if m > 0:
            pmm = -math.sqrt((2 * m + 1) / (2 * m)) * st * pmm
            cm, sm = cm * cp - sm * sp, sm * cp + cm * sp
        p2, p1 = torch.zeros_like(ct), pmm
        for l in range(m, L + 1):
            if l == m + 1:
                p2, p1 = p1, math.sqrt(2 * m + 3) * ct * p1
            elif l > m + 1:
                a = math.sqrt((4 * l * l - 1) / (l * l - m * m))
                b = math.sqrt(((l - 1) ** 2 - m * m) / (4 * (l - 1) ** 2 - 1))
                p2, p1 = p1, a * (ct * p1 - b * p2)
            if m == 0:
                yield l * l + l, p1
            else:
                yield l * l + l + m, math.sqrt(2) * p1 * cm
                yield l * l + l - m, math.sqrt(2) * p1 * sm


class _Obs:
    """The kernels K_j of a layout: deposits and force sums in 64 bits."""

    def __init__(self, lay, V=None, S=None):
        self.lay, self.V, self.S = lay, V, S
        alm = lay["dens"] == "alm"
        self.nlm = (lay["l_max"] + 1) ** 2 if alm else 1
        self.re = _log_edges(lay["r_min"], lay["r_max"], lay["n_r"] - 1 if alm else lay["n_r"])
        self.Re = _log_edges(lay["R_min"], lay["R_max"], lay["n_R"])
        self.nd = lay["n_r"] * self.nlm
        self.per = {"v2": 1, "gh": lay["gh_nmax"], "losvd": lay["n_v"]}[lay["kin"]]
        self.J = self.nd + lay["n_R"] * self.per
        if lay["kin"] == "losvd":
            self.ve = torch.linspace(lay["v_min"], lay["v_max"], lay["n_v"] + 1, dtype=F64, device="cuda")

    def entries(self, p):
        """(index or -1, value) of every kernel a particle may have."""
        lay, vz = self.lay, p["vz"]
        R = torch.sqrt(p["x"] ** 2 + p["y"] ** 2)
        r = torch.sqrt(R * R + p["z"] ** 2)
        k = _bin(r, self.re)
        if lay["dens"] == "alm":
            kk = k.clamp_min(0)
            g = (self.re[kk + 1] - r) / (self.re[kk + 1] - self.re[kk])
            for lm, Y in _harmonics(lay["l_max"], *_direction(p["x"], p["y"], p["z"])):
                yield torch.where(k >= 0, kk * self.nlm + lm, -1), g * Y
                yield torch.where(k >= 0, (kk + 1) * self.nlm + lm, -1), (1 - g) * Y
        else:
            yield k, torch.ones_like(r)
        a = _bin(R, self.Re)
        aa = a.clamp_min(0)
        base = self.nd + aa * self.per
        if lay["kin"] == "v2":
            yield torch.where(a >= 0, base, -1), vz * vz
        elif lay["kin"] == "losvd":
            b = _bin(vz, self.ve)
            yield torch.where((a >= 0) & (b >= 0), base + b, -1), torch.ones_like(vz)
        else:
            nu = (vz - self.V[aa]) / self.S[aa]
            g = math.sqrt(2) * torch.exp(-0.5 * nu * nu)
            h0, h1 = torch.ones_like(nu), math.sqrt(2) * nu
            for n in range(1, self.per + 1):
                yield torch.where(a >= 0, base + n - 1, -1), g * h1
                h0, h1 = h1, math.sqrt(2 / (n + 1)) * nu * h1 - math.sqrt(n / (n + 1)) * h0

    def deposit(self, p, w):
        y = torch.zeros(self.J + 1, dtype=F64, device="cuda")
        for j, k in self.entries(p):
            y += torch.bincount(torch.where(j >= 0, j, self.J), weights=w * k, minlength=self.J + 1)
        return y[: self.J]

    def gather(self, p, c):
        c = torch.cat([c, torch.zeros(1, dtype=F64, device="cuda")])
        return sum(c[j] * k for j, k in self.entries(p))  # index -1: the zero at the end


def _targets(case, pot, lay, n_model, g):
    """Y, sigma, V_p, sigma_p of a realization of another distribution function:
    2 % errors (5 % of LOSVD bins), floored at the model's own particle noise."""
    n = 1 << 17
    p = _model(case, pot, n, g, anisotropic=True)
    o = _Obs(lay)
    nR = lay["n_R"]
    a = _bin(torch.sqrt(p["x"] ** 2 + p["y"] ** 2), o.Re)
    a = torch.where(a >= 0, a, nR)
    m = torch.bincount(a, minlength=nR + 1)[:nR].clamp_min(1)
    S = torch.sqrt(torch.bincount(a, weights=p["vz"] ** 2, minlength=nR + 1)[:nR] / m).clamp_min(0.05)
    V = torch.zeros(nR, dtype=F64, device="cuda")
    o = _Obs(lay, V, S)
    Y = o.deposit(p, torch.full((n,), 1.0 / n, dtype=F64, device="cuda"))
    sig = torch.empty_like(Y)
    if lay["dens"] == "alm":
        a0 = Y[: o.nd].reshape(-1, o.nlm)[:, 0].abs()
        sig[: o.nd] = 0.02 * torch.maximum(a0, 1e-3 * a0.max()).repeat_interleave(o.nlm)
    else:
        a0 = Y[: o.nd].abs()
        sig[: o.nd] = 0.02 * torch.maximum(a0, 1e-3 * a0.max())
    rest = Y[o.nd:]
    if lay["kin"] == "v2":
        sig[o.nd:] = 0.02 * torch.maximum(rest, 1e-3 * rest.max())
    elif lay["kin"] == "gh":
        sig[o.nd:] = 0.02 * (m / n).repeat_interleave(o.per)
    else:
        h = rest.reshape(nR, -1)
        peak = torch.maximum(h.max(1, keepdim=True).values, 1e-4 * h.max())
        sig[o.nd:] = (0.05 * torch.maximum(h, 0.01 * peak)).reshape(-1)
    m1 = 1.0 / min(n_model, n)
    sig = torch.sqrt(sig * sig + 4 * (Y.abs() + m1) * m1)
    Y = Y + sig * torch.randn(o.J, generator=g, device="cuda", dtype=F64)
    return {"Y": Y, "sigma": sig, "V_p": V, "sigma_p": S}


# ------------------------------------------------------------- what is timed
def _sizes(case, g):
    """Particle counts of the fits: log-uniform over [n, n_hi] in a batch."""
    if case["kind"] != "batch":
        return [case["n"]]
    u = torch.rand(case["fits"], generator=g, device="cuda", dtype=F64).tolist()
    return [int(round(case["n"] * (case["n_hi"] / case["n"]) ** v)) for v in u]


def _inputs(case, seed):
    """What the fits of a case start from, one dict per fit: the same for the
    timed program and for the 64-bit reference. The sizes of a batch are the
    case's own; everything else comes from the seed."""
    g0 = torch.Generator(device="cuda").manual_seed(4)
    sizes = _sizes(case, g0)
    g = torch.Generator(device="cuda").manual_seed(int(seed))
    lay = _layout(case)
    for k, n in enumerate(sizes):
        pot = _potential(case, k, len(sizes))
        p = _rounded(_model(case, pot, n, g), case["dtype"])
        yield {"n": n, "pot": pot, "lay": lay, "par": _params(case, pot), "p": p,
               "T": _targets(case, pot, lay, n, g)}


class _State:
    def __init__(self):
        self.case, self.fits, self.batch, self.pos, self.vel = None, [], None, [], []
        self.V = self.S = None

    def __del__(self):
        if self.batch is not None:
            self.batch.close()


def prepare(case, seed):
    """The fits with their targets set, at the package's tuned launch; a batch
    has them admitted."""
    s = _State()
    s.case = case
    lay = _layout(case)
    mode = "batch" if case["kind"] == "batch" else "single"
    for d in _inputs(case, seed):
        if mode == "single":
            tuning.use("single", case["dtype"], lay, d["n"])
        f = Fit(d["pot"], d["lay"], d["par"], d["p"], dtype=case["dtype"])
        T = {k: v.cpu().numpy() for k, v in d["T"].items()}
        if case["kind"] == "observe":
            s.V, s.S = (T["V_p"], T["sigma_p"]) if case["kin"] == "gh" else (None, None)
        else:
            f.set_targets(T["Y"], T["sigma"], T["V_p"], T["sigma_p"])
        s.fits.append(f)
        # the three positions (velocities) of a fit as one (3, n) view of its state
        for a, b, to in (("x", "y", s.pos), ("vx", "vy", s.vel)):
            to.append(f.t[a].as_strided((3, d["n"]), (f.t[b].storage_offset() - f.t[a].storage_offset(), 1)))
    if mode == "batch":
        tuning.use("batch", case["dtype"], lay)
        s.batch = Batch(max_fits=len(s.fits))
        for f in s.fits:
            if not s.batch.admit(f, 1 << 30):
                raise RuntimeError("admission failed")
    return s


def run(state):
    case = state.case
    if case["kind"] == "observe":
        return {"y": state.fits[0].observe(state.V, state.S)}
    if case["kind"] == "batch":
        state.batch.run(case["steps"])
        out = {"u": [f.t["u"] for f in state.fits]}
        if len(state.fits) <= 16:
            out.update(pos=state.pos, vel=state.vel)
        return out
    f = state.fits[0]
    f.step(case["steps"])
    out = {"u": f.t["u"], "uh": f.t["uh"], "pos": state.pos[0], "vel": state.vel[0]}
    if case["monitor"]:
        out["obs"] = f.observables()
    return out


def work(case):
    """Particle state read and written once per pass, or once per step where it
    cannot stay on the chip; the operations of a step counted from its formulas."""
    g0 = torch.Generator(device="cuda").manual_seed(4)
    n = sum(_sizes(case, g0))
    b = 8 if case["dtype"] == "f64" else 4
    nlm = lambda l: (l + 1) ** 2 if l >= 0 else 0
    obs = 30 + 12 * nlm(case["alm"]) + {"v2": 4, "gh": 10 + 8 * case["gh"], "losvd": 6}[case["kin"]]
    if case["kind"] == "observe":
        return {"bytes": 5 * b * n, "flops": obs * n}
    per = 2 * obs + 45 + (25 if case["nfw"] else 0) + 30 * nlm(case["scf"])
    times = case["steps"] if 8 * b * n > ON_CHIP else 1
    return {"bytes": 15 * b * n * times, "flops": per * n * case["steps"]}


# ------------------------------------------------------- the reference, 64 bits
class _Multipole:
    """The stellar potential as a multipole expansion of the particles."""

    def __init__(self, par, c, p, u):
        self.L, self.K = par["scf_lmax"], par["scf_nr"]
        rho = _log_edges(par["scf_rmin"], par["scf_rmax"], self.K - 1)
        self.rho, self.h = rho, math.log(par["scf_rmax"] / par["scf_rmin"]) / (self.K - 1)
        r = torch.sqrt(p["x"] ** 2 + p["y"] ** 2 + p["z"] ** 2)
        q = torch.bucketize(r, rho, right=True)
        self.val, self.der = {}, {}
        for lm, Y in _harmonics(self.L, *_direction(p["x"], p["y"], p["z"])):
            l = int(math.isqrt(lm))
            A = torch.bincount(q, weights=u * r ** l * Y, minlength=self.K + 1)
            B = torch.bincount(q, weights=u * r ** -(l + 1) * Y, minlength=self.K + 1)
            a, b = A.cumsum(0)[: self.K], B.flip(0).cumsum(0).flip(0)[1:]
            f = -4 * math.pi * c / (2 * l + 1)
            self.val[lm] = f * (rho ** -(l + 1) * a + rho ** l * b)
            self.der[lm] = f * (-(l + 1) * rho ** -(l + 1) * a + l * rho ** l * b)

    def accel(self, x, y, z):
        X = [v.detach().clone().requires_grad_(True) for v in (x, y, z)]
        with torch.enable_grad():
            r = torch.sqrt(X[0] ** 2 + X[1] ** 2 + X[2] ** 2)
            q = torch.bucketize(r.detach(), self.rho, right=True)
            lo, hi = (q - 1).clamp(0, self.K - 1), q.clamp(0, self.K - 1)
            t = ((torch.log(r) - math.log(float(self.rho[0]))) / self.h - (q - 1)).clamp(0, 1)
            inside, outside = q == 0, q == self.K
            v = r / torch.where(inside, self.rho[0], self.rho[-1])
            total = torch.zeros((), dtype=F64, device="cuda")
            for lm, Y in _harmonics(self.L, *_direction(*X)):
                l = int(math.isqrt(lm))
                P0, D0, P1, D1 = self.val[lm][lo], self.der[lm][lo], self.val[lm][hi], self.der[lm][hi]
                f = ((2 * t ** 3 - 3 * t ** 2 + 1) * P0 + self.h * (t ** 3 - 2 * t ** 2 + t) * D0
                     + (3 * t ** 2 - 2 * t ** 3) * P1 + self.h * (t ** 3 - t ** 2) * D1)
                core = v ** l * (P1 + (D1 - l * P1) * (v * v - 1) / 2)
                w = 1 / v
                far = w ** (l + 1) * (P0 + (-D0 - (l + 1) * P0) * (w * w - 1) / 2)
                total = total + (torch.where(inside, core, torch.where(outside, far, f)) * Y).sum()
            return tuple(-d for d in torch.autograd.grad(total, X))


def _cells(P, par, p):
    """Cell of every particle on the (E, L / L_c) grid."""
    x, y, z, vx, vy, vz = (p[k] for k in FIELDS)
    r = torch.sqrt(x * x + y * y + z * z)
    E = 0.5 * (vx * vx + vy * vy + vz * vz) - P.gm / (r + P.a)
    if P.gn:
        E = E - P.gn * torch.log1p(r / P.rs) / r
    if P.v2:
        E = E + 0.5 * P.v2 * torch.log(P.r02 + x * x + y * y + z * z * P.iq2)
    lx, ly, lz = y * vz - z * vy, z * vx - x * vz, x * vy - y * vx
    L = torch.sqrt(lx * lx + ly * ly + lz * lz)
    rt = torch.logspace(-8, 14 if not P.v2 else 4, 1 << 16, dtype=F64, device="cuda")
    Et = P.phi(rt) + 0.5 * P.vc2(rt)
    i = (torch.bucketize(E, Et, right=True) - 1).clamp(0, rt.numel() - 2)
    rc = torch.exp(torch.lerp(torch.log(rt[i]), torch.log(rt[i + 1]), ((E - Et[i]) / (Et[i + 1] - Et[i])).clamp(0, 1)))
    for _ in range(3):  # Newton steps on E_c(r) = E, in ln r
        d = 0.5 * P.mass(rc) / rc + P.gm * P.a * rc / (rc + P.a) ** 3
        if P.gn:
            d = d + 0.5 * P.gn * rc / (P.rs ** 2 * (1 + rc / P.rs) ** 2)
        if P.v2:
            d = d + P.v2 * rc ** 2 * (2 * P.r02 + rc ** 2) / (P.r02 + rc ** 2) ** 2
        rc = rc * torch.exp(-((P.phi(rc) + 0.5 * P.vc2(rc) - E) / d).clamp(-1, 1))
    xc = L / (rc * torch.sqrt(P.vc2(rc)))
    phi0 = P.phi(torch.zeros(1, dtype=F64, device="cuda"))
    if not P.v2:
        xc = torch.where(E < 0, xc, 0.0)
    xc = torch.where(E > phi0, xc, 1.0)
    e, lo, hi = (torch.exp(E), math.exp(par["E_lo"]), math.exp(par["E_hi"])) if par["cells"] & 2 else (E, par["E_lo"], par["E_hi"])
    k = ((e - lo) * (par["n_E"] / (hi - lo))).clamp(0, par["n_E"] - 1).long()
    c = k * par["n_x"] + (xc * par["n_x"]).clamp(0, par["n_x"] - 1).long()
    return torch.where(lz < 0, c + par["n_E"] * par["n_x"], c) if par["cells"] & 1 else c


def _smoothed(w0, par):
    """The thin-plate smoothed prior grid, lambda by generalized cross validation."""
    nE, nx = par["n_E"], par["n_x"]
    hE, hx = (par["E_hi"] - par["E_lo"]) / nE, 1.0 / nx

    def second(n, h):
        D = np.zeros((max(n - 2, 0), n))
        for k in range(n - 2):
            D[k, k:k + 3] = np.array([1.0, -2.0, 1.0]) / h ** 2
        return D

    d2E, d2x = second(nE, hE), second(nx, hx)
    dE, dx = np.diff(np.eye(nE), axis=0) / hE, np.diff(np.eye(nx), axis=0) / hx
    P = np.kron(d2E.T @ d2E, np.eye(nx)) + 2 * np.kron(dE.T @ dE, dx.T @ dx) + np.kron(np.eye(nE), d2x.T @ d2x)
    g, Q = np.linalg.eigh(P)
    g[:3] = 0.0
    w = w0.cpu().numpy()
    wh = Q.T @ w

    def gcv(p):
        t = 10.0 ** p * g
        f = t / (1 + t)
        return np.mean((f * wh) ** 2) / np.mean(f) ** 2

    ghi = 4 / hE ** 2 + 4 / hx ** 2
    glo = min(4 * math.sin(math.pi / (2 * n)) ** 2 / h ** 2 for n, h in ((nE, hE), (nx, hx)))
    lo, hi = -2 * math.log10(ghi) - 4, -2 * math.log10(glo) + 4
    k1 = int((hi - lo) / 0.25) + 1
    i = int(np.argmin([gcv(lo + 0.25 * k) for k in range(k1)]))
    a, b = lo + 0.25 * max(i - 1, 0), lo + 0.25 * min(i + 1, k1 - 1)
    for last in (False, True):
        i = int(np.argmin([gcv(a + (b - a) * k / 64) for k in range(65)]))
        if last:
            lam = 10.0 ** (a + (b - a) * i / 64)
        a, b = a + (b - a) * max(i - 1, 0) / 64, a + (b - a) * min(i + 1, 64) / 64
    v = Q @ (wh / (1 + lam * g))
    return torch.tensor(np.maximum(v, 1e-3 * w.mean()), dtype=F64, device="cuda")


def _reference(d, steps):
    """`steps` M2M steps of one fit in 64 bits."""
    par, P, T, n = d["par"], _Pot(d["pot"]), d["T"], d["n"]
    o = _Obs(d["lay"], T["V_p"], T["sigma_p"])
    p = {k: v.to(F64) for k, v in d["p"].items()}
    u, uh = torch.ones(n, dtype=F64, device="cuda"), torch.ones(n, dtype=F64, device="cuda")
    dt, w0 = par["dt"], par["mass"] / n
    scf = par.get("scf_nr", 0) > 0
    field = _Multipole(par, d["pot"]["G"] * d["pot"]["upsilon"] * w0, p, u) if scf else None
    q = -math.expm1(-par["alpha"] * dt)
    y = o.deposit(p, u * w0)
    yt = y.clone()
    prior = torch.ones(par["n_E"] * par["n_x"] * (2 if par["cells"] & 1 else 1), dtype=F64, device="cuda")
    cells = None
    for k in range(steps):
        if cells is not None:
            uh, cells = prior[cells], None
        chi = o.gather(p, par["eps"] * dt * w0 * (yt - T["Y"]) / T["sigma"] ** 2)
        gwr = 1.0 if par["entropy"] == "gwr" else 0.0
        u = u * torch.exp(-par["eps"] * dt * par["mu"] * (torch.log(u / uh) + gwr) - chi)
        for a, b in zip(FIELDS[:3], FIELDS[3:]):
            p[a] = p[a] + 0.5 * dt * p[b]
        acc = P.accel(p["x"], p["y"], p["z"], stars=not scf)
        if scf:
            acc = [a + b for a, b in zip(acc, field.accel(p["x"], p["y"], p["z"]))]
        for a, b, f in zip(FIELDS[:3], FIELDS[3:], acc):
            p[b] = p[b] + dt * f
            p[a] = p[a] + 0.5 * dt * p[b]
        y = o.deposit(p, u * w0)
        yt = yt + q * (y - yt)
        if scf and (k + 1) % par["scf_every"] == 0:
            field = _Multipole(par, d["pot"]["G"] * d["pot"]["upsilon"] * w0, p, u)
        if par["entropy"] == "mpr" and (k + 1) % par["prior_every"] == 0:
            cells = _cells(P, par, p)
            cnt = torch.bincount(cells, minlength=prior.numel())
            mean = torch.bincount(cells, weights=u, minlength=prior.numel()) / cnt.clamp_min(1)
            prior = torch.where(cnt > 0, mean, prior)
            if par["smooth"]:
                prior = _smoothed(prior, par)
    delta = (yt - T["Y"]) / T["sigma"]
    return {"u": u, "uh": uh, "pos": torch.stack([p[k] for k in FIELDS[:3]]),
            "vel": torch.stack([p[k] for k in FIELDS[3:]]),
            "obs": {"y": y, "ytilde": yt, "delta": delta, "chi2": float((delta * delta).sum())}}


def exact(case, seed):
    with torch.no_grad():
        if case["kind"] == "observe":
            d = next(_inputs(case, seed))
            w = torch.full((d["n"],), 1.0 / d["n"], dtype=F64, device="cuda")
            y = _Obs(d["lay"], d["T"]["V_p"], d["T"]["sigma_p"]).deposit({k: v.to(F64) for k, v in d["p"].items()}, w)
            return {"y": y}
        got = []
        for d in _inputs(case, seed):
            r = _reference(d, case["steps"])
            got.append(r)
    if case["kind"] == "batch":
        return {k: [r[k] for r in got] for k in (("u", "pos", "vel") if len(got) <= 16 else ("u",))}
    if not case["monitor"]:
        del got[0]["obs"]
    return got[0]
