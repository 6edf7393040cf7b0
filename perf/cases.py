"""The work that users of the library have it do, as timed cases.

Kinds of case (each through the public entry points of paper_1703_00879_amd):

* ``mock``: one mock catalogue from its parameters and seed: cola_make_ic, then cola_step to
  z = 0 (the final displacements and velocities come back);
* ``ic``: the 2LPT initial conditions alone, cola_make_ic (a run that is stepped elsewhere, or
  whose first output is its initial state);
* ``force``: cola_pm_force on particles in hand (a force evaluation inside another
  integrator, or the mesh fields of a snapshot);
* ``pk``: cola_power_spectrum of particles in hand (the summary statistic of a snapshot);
* ``ensemble``: uneven small mocks stepped together as captured graphs (Ensemble.run).

``exact`` evaluates the method in 64 bits with plain torch and numpy.
"""

import math
import random

import numpy as np
import torch

from paper_1703_00879_amd import cola as C

DEV = "cuda:0"
OM, OB, H100, NS, S8, TCMB = 0.3, 0.05, 0.7, 0.96, 0.8, 2.7255
H0C = 1.0 / 2997.92458            # H0/c in h/Mpc
MODELS = {"lcdm": C.LCDM, "fr": C.FR_HS1, "ndgp": C.NDGP, "symmetron": C.SYMMETRON,
          "kmouflage": C.KMOUFLAGE}
FILTERS = {"gauss": C.SMOOTH_GAUSS, "tophat": C.SMOOTH_TOPHAT, "sharpk": C.SMOOTH_SHARPK}


def listed():
    return [
        # the smallest run in earnest: the parity configuration of f(R) with its own
        # scale-dependent growth, where launches and latency count
        {"name": "mock_fr5_32", "kind": "mock", "model": "fr", "fr0": 1e-5, "np": 32, "ratio": 2,
         "spacing": 6.25, "steps": 10},
        # the smallest box of the ensembles, plain gravity
        {"name": "mock_lcdm_64", "kind": "mock", "model": "lcdm", "np": 64, "ratio": 2,
         "spacing": 2.0, "steps": 10},
        # a radix-3 box of the ensembles, Vainshtein screening on a smoothed density
        {"name": "mock_ndgp_96", "kind": "mock", "model": "ndgp", "rc": 1.0, "np": 96, "ratio": 2,
         "spacing": 2.0, "steps": 10},
        # an ordinary request of the serving mix: f(R), scale-dependent, 20 steps
        {"name": "mock_fr6_256", "kind": "mock", "model": "fr", "fr0": 1e-6, "np": 256, "ratio": 2,
         "spacing": 2.0, "steps": 20},
        # the largest: the nDGP configuration of 512^3 particles on a 1024^3 mesh, 10 steps
        {"name": "mock_ndgp_512", "kind": "mock", "model": "ndgp", "rc": 1.0, "np": 512, "ratio": 2,
         "spacing": 2.0, "steps": 10},
        # initial conditions of the largest (radix-3) run of the serving mix
        {"name": "ic_fr5_384", "kind": "ic", "model": "fr", "fr0": 1e-5, "np": 384, "ratio": 2,
         "spacing": 2.0, "steps": 30},
        # forces on a late, clustered f(R) snapshot as the 1024^3 mesh of a large run takes them
        {"name": "force_fr5_512", "kind": "force", "model": "fr", "fr0": 1e-5, "np": 512, "ratio": 2,
         "spacing": 2.0, "a": 0.95, "rms": 5.0, "clustered": True},
        # forces and all five meshes of a gradient-screened model on a radix-3 mesh
        {"name": "force_km_192_meshes", "kind": "force", "model": "kmouflage", "np": 192, "ratio": 2,
         "spacing": 2.0, "a": 0.8, "rms": 4.0, "clustered": True, "meshes": True},
        # P(k) of a mid-size box, early (unclustered), and of the largest, late
        {"name": "pk_128", "kind": "pk", "np": 128, "ratio": 2, "spacing": 2.0, "rms": 0.5,
         "clustered": False},
        {"name": "pk_512", "kind": "pk", "np": 512, "ratio": 2, "spacing": 2.0, "rms": 5.0,
         "clustered": True},
        # twelve uneven boxes of mixed models stepped together
        {"name": "ensemble_12", "kind": "ensemble", "members": 12, "mix": 4, "np_max": 192,
         "steps": 10},
    ]


GRIDS = [16, 24, 32, 48, 64, 96, 128, 192, 256, 384, 512]


def draw(rng):
    kind = rng.choices(["mock", "ic", "force", "pk", "ensemble"], [4, 1, 3, 2, 1])[0]
    if kind == "ensemble":
        top = rng.choice([64, 96, 128, 192])
        return {"kind": kind, "members": rng.randint(3, 8 if top == 192 else 16),
                "mix": rng.randrange(1000), "np_max": top, "steps": rng.randint(5, 12)}
    model = rng.choice(["lcdm", "fr", "fr", "ndgp", "ndgp"])
    if kind == "force":
        model = rng.choice([model, "symmetron", "kmouflage"])
    # ratio 2 is what runs take; 1, 3 and 4 are the other mesh refinements the library has
    ratio = rng.choice([2, 2, 2, 2, 1, 4, 3])
    if ratio == 3:
        np1d = rng.choice([16, 32, 64, 128, 256])
    else:
        np1d = rng.choice([g for g in GRIDS if g * ratio <= 1024 and g <= 384])
    c = {"kind": kind, "model": model, "np": np1d, "ratio": ratio,
         "spacing": round(rng.uniform(0.8, 6.5), 2)}
    if model == "fr":
        c["fr0"] = rng.choice([1e-6, 1e-5, 1e-4])
    if model == "ndgp":
        c["rc"] = rng.choice([0.5, 1.0])
        c["filter"] = rng.choice(["gauss", "gauss", "tophat", "sharpk"])
    if model != "lcdm":
        c["screening"] = rng.random() < 0.85
    if kind in ("mock", "ic"):
        most = 8 if np1d * ratio > 512 else 30
        c["steps"] = rng.randint(3, most)
        if model == "fr":
            c["lcdm_growth"] = rng.random() < 0.25   # ΛCDM growth factors, modified force
    else:
        c["rms"] = round(rng.uniform(0.1, 6.0), 2)   # displacement, in mesh cells per axis
        c["clustered"] = rng.random() < 0.6
    if kind == "force":
        c["a"] = round(rng.uniform(0.1, 1.0), 3)
        c["meshes"] = np1d * ratio <= 512 and rng.random() < 0.4
    if kind == "pk":
        c["nbins"] = rng.choice([0, max(1, np1d * ratio // 3)])   # 0: the default, n_mesh / 2
    return c


# ----------------------------------------------------------------------------- inputs
def params_of(c, seed):
    return C.Params(model=MODELS[c.get("model", "lcdm")], fr0_abs=c.get("fr0", 1e-5),
                    rc_h0=c.get("rc", 1.0), filter=FILTERS[c.get("filter", "gauss")],
                    screening=int(c.get("screening", True)),
                    growth_mode=int(c.get("lcdm_growth", False)), np1d=c["np"],
                    nmesh1d=c["np"] * c["ratio"], box=c["np"] * c["spacing"],
                    n_steps=c.get("steps", 2), seed=1000 + seed, omega_m=OM, omega_b=OB, h=H100,
                    n_s=NS, sigma8=S8, t_cmb=TCMB, z_init=19.0)


def members_of(c, seed):
    """The ensemble's runs: uneven grids up to np_max and mixed models."""
    r = random.Random(c["mix"])
    grids = [g for g in (64, 96, 128, 192) if g <= c["np_max"]]
    out = []
    for j in range(c["members"]):
        m = {"np": r.choice(grids), "ratio": 2, "spacing": 2.0, "steps": c["steps"]}
        m.update(r.choice([{"model": "lcdm"}, {"model": "fr", "fr0": 1e-6},
                           {"model": "fr", "fr0": 1e-5}, {"model": "fr", "fr0": 1e-4},
                           {"model": "ndgp", "rc": 0.5}, {"model": "ndgp", "rc": 1.0}]))
        out.append((m, seed * 100 + j))
    return out


def displacements(c, seed):
    """u [3][N] float32 in Mpc/h: the gradient of a Gaussian field with a steep spectrum,
    `rms` cells per axis, as an evolved box has it; with `clustered` every fourth particle is
    pulled into one of 64 small clumps, as the halos of a late snapshot."""
    n, cell = c["np"], c["spacing"] / c["ratio"]
    g = torch.Generator(device=DEV)
    g.manual_seed(7919 * seed + 17)
    wk = torch.fft.rfftn(torch.randn((n, n, n), generator=g, device=DEV))
    nu = freqs(n, torch.float32)
    k2 = nu[0] ** 2 + nu[1] ** 2 + nu[2] ** 2
    k2[0, 0, 0] = 1.0
    wk *= k2 ** -1.4
    wk[0, 0, 0] = 0.0
    u = torch.empty((3, n ** 3), device=DEV)
    for a in range(3):
        u[a] = torch.fft.irfftn(1j * nu[a] * wk, s=(n, n, n)).reshape(-1)
    u *= c["rms"] * cell / u.square().mean().sqrt()
    if c["clustered"]:
        N, L = n ** 3, n * c["spacing"]
        pick = torch.rand(N, generator=g, device=DEV) < 0.25
        which = torch.randint(0, 64, (N,), generator=g, device=DEV)
        for a, q in enumerate(lattice(n)):
            centre = torch.rand(64, generator=g, device=DEV) * L
            d = centre[which] + torch.randn(N, generator=g, device=DEV) * (0.8 * cell)
            d -= q.float() * c["spacing"] + 0.5 * cell
            d -= L * torch.round(d / L)
            u[a] = torch.where(pick, d, u[a])
    return u


def prepare(case, seed):
    if case["kind"] == "ensemble":
        runs = [params_of(m, s) for m, s in members_of(case, seed)]
        return {"kind": "ensemble", "ps": runs, "sts": [C.State(p, device=DEV) for p in runs]}
    p = params_of(case, seed)
    st = C.State(p, device=DEV)
    s = {"kind": case["kind"], "p": p, "st": st, "steps": case.get("steps", 0)}
    if case["kind"] in ("force", "pk"):
        C.cola_prepare(p, st)
        st.disp_f.copy_(displacements(case, seed))
        st.vel_f.zero_()
    if case["kind"] == "force":
        s["a"] = case["a"]
        s["force"] = torch.empty((3, p.np1d ** 3), device=DEV)
        s["meshes"] = torch.empty((5,) + (p.nmesh1d,) * 3, device=DEV) if case.get("meshes") else None
    if case["kind"] == "pk":
        s["nbins"] = case.get("nbins") or None
    return s


def run(s):
    if s["kind"] == "ensemble":
        for p, st in zip(s["ps"], s["sts"]):
            C.cola_make_ic(p, st)
        e = C.Ensemble(s["ps"], s["sts"])
        e.run(8)
        e.close()
        return [st.disp_f for st in s["sts"]]
    p, st = s["p"], s["st"]
    if s["kind"] == "mock":
        C.cola_make_ic(p, st)
        for i in range(s["steps"]):
            C.cola_step(p, st, i)
        return {"u": st.disp_f, "v": st.vel_f}
    if s["kind"] == "ic":
        C.cola_make_ic(p, st)
        return {"u": st.disp_f}
    if s["kind"] == "force":
        C.cola_pm_force(p, st, s["a"], s["force"], s["meshes"])
        out = {"force": s["force"]}
        if s["meshes"] is not None:
            out.update(zip(("rho", "src", "fx", "fy", "fz"), s["meshes"]))
        return out
    k, P, n = C.cola_power_spectrum(p, st, s["nbins"])
    return {"k": k, "P": P, "n": n}


# ----------------------------------------------------------------------------- least work
def work(case):
    """Particle state read and written once a step (u, v and the two LPT terms in, u and v
    out; 72 bytes a particle), spectra and meshes that are asked for, and 5/2 n log2 n flops
    per real transform of n values."""
    if case["kind"] == "ensemble":
        w = [work(dict(m, kind="mock")) for m, _ in members_of(case, 0)]
        return {"bytes": sum(x["bytes"] for x in w), "flops": sum(x["flops"] for x in w)}
    N = case["np"] ** 3
    M = (case["np"] * case["ratio"]) ** 3
    mesh_fft, part_fft = 2.5 * M * math.log2(M), 2.5 * N * math.log2(N)
    screened = case.get("model", "lcdm") != "lcdm" and case.get("screening", True)
    per_force = (6 if screened else 4) * mesh_fft
    kdep = case.get("model") == "fr" and not case.get("lcdm_growth")
    ic = {"bytes": 24.0 * N + (8.0 if kdep else 24.0) * N, "flops": (9 + (3 if kdep else 6)) * part_fft}
    if case["kind"] == "ic":
        return ic
    if case["kind"] == "mock":
        s = case["steps"]
        return {"bytes": ic["bytes"] + s * 72.0 * N,
                "flops": ic["flops"] + s * (per_force + (6 * part_fft if kdep else 0))}
    if case["kind"] == "force":
        return {"bytes": 24.0 * N + (20.0 * M if case.get("meshes") else 0.0), "flops": per_force}
    return {"bytes": 12.0 * N, "flops": mesh_fft}


# ----------------------------------------------------------------------------- 64-bit values
F64 = torch.float64


def lattice(n):
    """Lattice indices (ix, iy, iz) of the particles in their stored order."""
    p = torch.arange(n ** 3, device=DEV)
    return p // (n * n), (p // n) % n, p % n


def freqs(n, dtype=F64):
    """Integer frequencies per axis, shaped to broadcast; the odd-derivative convention zeroes
    each axis's Nyquist plane (see grad)."""
    full = torch.fft.fftfreq(n, d=1.0 / n, device=DEV, dtype=dtype)
    half = torch.arange(n // 2 + 1, device=DEV, dtype=dtype)
    return full[:, None, None], full[None, :, None], half[None, None, :]


def grad(n, L):
    """k_c per axis, zero on that axis's Nyquist plane."""
    return [torch.where(nu.abs() == n // 2, torch.zeros_like(nu), nu) * (2 * math.pi / L)
            for nu in freqs(n)]


def k_squared(n, L):
    nu = freqs(n)
    return (nu[0] ** 2 + nu[1] ** 2 + nu[2] ** 2) * (2 * math.pi / L) ** 2


def inverse(x):
    """1/x, zero where x is zero."""
    r = x.reciprocal()
    return torch.where(x == 0, torch.zeros_like(r), r)


def back(fk, n):
    return torch.fft.irfftn(fk, s=(n, n, n))


def hubble(a):
    return math.sqrt(OM / a ** 3 + 1 - OM)


def model_at(c, a):
    """(a^2 m^2, C, screening scalar) of the fifth force at scale factor a."""
    m, ol = c.get("model", "lcdm"), 1 - OM
    if m == "fr":
        X, Y = OM / a ** 3 + 4 * ol, OM + 4 * ol
        fR = c["fr0"] * (Y / X) ** 2
        return a * a * H0C ** 2 * Y * (X / Y) ** 3 / (2 * c["fr0"]), 1 / 3, 1.5 * fR * a * a / H0C ** 2
    if m == "ndgp":
        E = hubble(a)
        beta = 1 + 2 * c["rc"] * E * (1 - 0.5 * OM / a ** 3 / E ** 2)
        return 0.0, 1 / (3 * beta), 8 * c["rc"] ** 2 * OM / (9 * beta ** 2 * a ** 3)
    if m == "symmetron":   # beta_* = 1, m_* = 2997.92458 H0, a_* = 0.5
        s = max(0.0, 1 - (0.5 / a) ** 3)
        thr = 3 * OM / (0.5 ** 3 * 2997.92458 ** 2) * a * a / H0C ** 2
        return a * a * H0C ** 2 * 2997.92458 ** 2 * s, 2 * s, thr
    if m == "kmouflage":   # beta = 0.5, K0 = 1, m = 3, lambda = 1e6 Mpc/h
        return 0.0, 2 * 0.5 ** 2, (1e6 * H0C ** 2 / a ** 2) ** 2
    return 0.0, 0.0, 0.0


def kmouflage_eps(R):
    """min(1, 1/P_X(X)) with P_X = 1 + 3 X^2 and P_X^2 X = R, by bisection in X."""
    lo, hi = torch.zeros_like(R), R.clone()
    for _ in range(200):
        mid = 0.5 * (lo + hi)
        up = (1 + 3 * mid * mid) ** 2 * mid < R
        lo, hi = torch.where(up, mid, lo), torch.where(up, hi, mid)
    return 1 / (1 + 3 * lo * lo)


def smoothing(k, name):
    """Window of radius 1 Mpc/h."""
    if name == "gauss":
        return torch.exp(-0.5 * k * k)
    if name == "sharpk":
        return (k <= 1).to(F64)
    x = torch.where(k == 0, torch.ones_like(k), k)
    w = torch.where(x < 0.1, 1 - x ** 2 / 10 + x ** 4 / 280 - x ** 6 / 15120 + x ** 8 / 1330560,
                    3 * (torch.sin(x) - x * torch.cos(x)) / x ** 3)
    return torch.where(k == 0, torch.ones_like(k), w)


class Cic:
    """Cloud-in-cell corners of the particles q + u on the mesh."""

    def __init__(self, c, u):
        self.n = c["np"] * c["ratio"]
        cell = c["spacing"] / c["ratio"]
        self.i, self.d = [], []
        for a, q in enumerate(lattice(c["np"])):
            f = 0.5 + u[a].to(F64) / cell
            self.d.append(f - torch.floor(f))
            self.i.append((q * c["ratio"] + torch.floor(f).long()) % self.n)

    def corners(self):
        for o in range(8):
            b = (o & 1, o >> 1 & 1, o >> 2)
            x, y, z = ((i + t) % self.n for i, t in zip(self.i, b))
            w = 1.0
            for d, t in zip(self.d, b):
                w = w * (d if t else 1 - d)
            yield (x * self.n + y) * self.n + z, w

    def deposit(self, mass):
        rho = torch.zeros(self.n ** 3, dtype=F64, device=DEV)
        for at, w in self.corners():
            rho.scatter_add_(0, at, w * mass)
        return rho.reshape((self.n,) * 3)

    def gather(self, field):
        out = 0
        for at, w in self.corners():
            out = out + w * field.reshape(-1)[at]
        return out


def pm_exact(c, u, a, meshes=False):
    """Per-particle PM force at a, and the five meshes if asked for."""
    n, L = c["np"] * c["ratio"], c["np"] * c["spacing"]
    cic = Cic(c, u)
    delta = cic.deposit(float(c["ratio"] ** 3)) - 1
    kap = 1.5 * OM * a
    a2m2, coupling, scr = model_at(c, a)
    k2 = k_squared(n, L)
    dk = torch.fft.rfftn(delta)
    tot = -kap * dk * inverse(k2)
    S, m = delta, c.get("model", "lcdm")
    if m != "lcdm":
        if c.get("screening", True):
            if m in ("fr", "symmetron"):
                phi = back(tot, n).abs()
                S = torch.where(phi > scr, delta * scr / phi, delta)
            elif m == "ndgp":
                W = smoothing(k2.sqrt(), c.get("filter", "gauss"))
                W[0, 0, 0] = 0.0
                x = scr * back(dk * W, n).clamp(min=-1.0)
                S = delta * 2 / (1 + torch.sqrt(1 + x))
            else:
                R = sum(back(-1j * kc * tot, n) ** 2 for kc in grad(n, L)) * scr
                S = delta * kmouflage_eps(R)
        del dk
        tot = tot - coupling * kap * torch.fft.rfftn(S) * inverse(k2 + a2m2 if a2m2 else k2)
    tot[0, 0, 0] = 0.0
    F, fm = [], []
    for kc in grad(n, L):
        f = back(-1j * kc * tot, n)
        F.append(cic.gather(f))
        if meshes:
            fm.append(f)
    return torch.stack(F), ([delta + 1, S] + fm if meshes else None)


def growth_exact(c, a_out):
    """(D1, D1'', D2, D2'') at a_out per integer |nu|^2 (one entry if growth has no scale)."""
    kdep = c.get("model") == "fr" and not c.get("lcdm_growth")
    m = "lcdm" if c.get("lcdm_growth") else c.get("model", "lcdm")
    if kdep:
        n2 = torch.arange(3 * (c["np"] // 2) ** 2 + 1, device=DEV, dtype=F64)
        kk = n2 * (2 * math.pi / (c["np"] * c["spacing"])) ** 2
    else:
        kk = torch.zeros(1, device=DEV, dtype=F64)

    def coeff(a):
        kap, E = 1.5 * OM * a, hubble(a)
        if m == "fr":
            a2m2 = model_at(c, a)[0]
            X, Y = OM / a ** 3 + 4 * (1 - OM), OM + 4 * (1 - OM)
            c0 = X ** 3 / (2 * c["fr0"] * Y ** 2)
            q = kk / (a * H0C) ** 2
            g2 = (-9 * OM ** 2 / (48 * a ** 6 * c["fr0"] ** 2) * kk / (a * H0C * E) ** 2
                  * X ** 5 / Y ** 4 / ((q + c0) * (0.5 * q + c0) ** 2))
            return kap * (1 + kk / (3 * (kk + a2m2))), 2 * a ** 4 * E * E * g2
        if m == "ndgp":
            beta = 1 / (3 * model_at(c, a)[1])
            g2 = -(c["rc"] * OM) ** 2 / (6 * E * E * beta ** 3 * a ** 6)
            return kap * (1 + 1 / (3 * beta)), 2 * a ** 4 * E * E * g2
        return kap, 0.0

    def rhs(lna, y):
        a = math.exp(lna)
        q, g = coeff(a)
        f = 1 / (a * a * hubble(a))
        return torch.stack([y[1] * f, q * y[0] * f, y[3] * f, (q * y[2] - (q + g) * y[0] ** 2) * f])

    a0 = a_out[0]
    g0 = a0 * a0 * hubble(a0)
    one = torch.ones_like(kk)
    y = torch.stack([one, g0 * one, -3 / 7 * one, -6 / 7 * g0 * one])
    lna, out = math.log(a0), []
    for a in a_out:
        n = max(1, math.ceil((math.log(a) - lna) / 5e-3))
        h = (math.log(a) - lna) / n
        for j in range(n if h > 0 else 0):
            t = lna + j * h
            k1 = rhs(t, y)
            k2 = rhs(t + h / 2, y + h / 2 * k1)
            k3 = rhs(t + h / 2, y + h / 2 * k2)
            k4 = rhs(t + h, y + h * k3)
            y = y + h / 6 * (k1 + 2 * k2 + 2 * k3 + k4)
        lna = math.log(a)
        q, g = coeff(a)
        out.append((y[0], q * y[0], y[2], q * y[2] - (q + g) * y[0] ** 2))
    return out, kdep


def white_noise(n, seed):
    """SplitMix64 counter stream and Box-Muller, on two's-complement 64-bit integers."""
    def u(j):
        def shr(z, b):
            return (z >> b) & ((1 << (64 - b)) - 1)

        def s64(x):
            return x - (1 << 64) if x >= 1 << 63 else x
        z = (j + 1) * s64(0x9E3779B97F4A7C15) + seed
        z = (z ^ shr(z, 30)) * s64(0xBF58476D1CE4E5B9)
        z = (z ^ shr(z, 27)) * s64(0x94D049BB133111EB)
        z = z ^ shr(z, 31)
        return (shr(z, 11).to(F64) + 0.5) * 2.0 ** -53
    j = 2 * torch.arange(n ** 3, device=DEV)
    return (torch.sqrt(-2 * torch.log(u(j))) * torch.cos(2 * math.pi * u(j + 1))).reshape(n, n, n)


def spectrum(k, xp):
    """k^ns T^2 with the Eisenstein-Hu no-wiggle transfer function; xp: numpy or torch."""
    om, ob, fb = OM * H100 ** 2, OB * H100 ** 2, OB / OM
    s = 44.5 * math.log(9.83 / om) / math.sqrt(1 + 10 * ob ** 0.75)
    al = 1 - 0.328 * math.log(431 * om) * fb + 0.38 * math.log(22.3 * om) * fb * fb
    gam = OM * H100 * (al + (1 - al) / (1 + (0.43 * k * H100 * s) ** 4))
    q = k * (TCMB / 2.7) ** 2 / gam
    L0 = xp.log(2 * math.e + 1.8 * q)
    T = L0 / (L0 + (14.2 + 731 / (1 + 62.5 * q)) * q * q)
    return k ** NS * T * T


class Lpt:
    """phi1_k and phi2_k on the particle grid, and the displacement fields they give."""

    def __init__(self, c, seed):
        n, L = c["np"], c["np"] * c["spacing"]
        self.n, self.k = n, grad(n, L)
        lnk = np.linspace(math.log(1e-5), math.log(1e2), 400001)
        k = np.exp(lnk)
        x = 8 * k
        W = np.where(x > 1e-2, 3 * (np.sin(x) - x * np.cos(x)) / x ** 3, 1 - x * x / 10)
        A = S8 ** 2 / np.trapezoid(k ** 3 * spectrum(k, np) * W * W / (2 * math.pi ** 2), lnk)
        d1 = growth_exact({"model": "lcdm"}, [0.05, 1.0])[0][1][0].item()
        k2 = k_squared(n, L)
        amp = torch.sqrt(n ** 3 / L ** 3 * A / d1 ** 2 * spectrum(k2.sqrt(), torch)) * inverse(k2)
        amp[0, 0, 0] = 0.0
        self.phi1 = amp * torch.fft.rfftn(white_noise(n, 1000 + seed))
        kk = [2 * math.pi / L * nu for nu in freqs(n)]
        h = [back(-kc * kc * self.phi1, n) for kc in kk]
        S = h[0] * h[1] + h[0] * h[2] + h[1] * h[2]
        del h
        for i, j in ((0, 1), (0, 2), (1, 2)):
            S -= back(-self.k[i] * self.k[j] * self.phi1, n) ** 2
        self.phi2 = -torch.fft.rfftn(S) * inverse(k2)
        nu = freqs(n)
        self.n2 = (nu[0] ** 2 + nu[1] ** 2 + nu[2] ** 2).long()

    def field(self, x1, x2, kdep):
        if kdep:
            g = x1[self.n2] * self.phi1 + x2[self.n2] * self.phi2
        else:
            g = x1 * self.phi1 + x2 * self.phi2
        return torch.stack([back(1j * kc * g, self.n).reshape(-1) for kc in self.k])


def tau(a0, a1):
    """int da / (a^3 E), Gauss-Legendre."""
    if a0 == a1:
        return 0.0
    x, w = np.polynomial.legendre.leggauss(100)
    l0, l1 = math.log(a0), math.log(a1)
    a = np.exp(0.5 * (l0 + l1) + 0.5 * (l1 - l0) * x)
    return float(0.5 * (l1 - l0) * np.sum(w / (a * a * np.sqrt(OM / a ** 3 + 1 - OM))))


def mock_exact(c, seed, steps):
    ai = 0.05
    a = [ai + i * (1 - ai) / c["steps"] for i in range(c["steps"] + 1)]
    lpt = Lpt(c, seed)
    G, kdep = growth_exact(c, a[:steps + 1])
    u = lpt.field(G[0][0], G[0][2], kdep)
    v = torch.zeros_like(u)
    for i in range(steps):
        F, _ = pm_exact(c, u, a[i])
        lo = a[0] if i == 0 else 0.5 * (a[i - 1] + a[i])
        v += tau(lo, 0.5 * (a[i] + a[i + 1])) * (F - lpt.field(G[i][1], G[i][3], kdep))
        u += tau(a[i], a[i + 1]) * v + lpt.field(G[i + 1][0] - G[i][0], G[i + 1][2] - G[i][2], kdep)
    return u, v


def pk_exact(c, seed):
    n, L = c["np"] * c["ratio"], c["np"] * c["spacing"]
    nbins = c.get("nbins") or n // 2
    dk = torch.fft.rfftn(Cic(c, displacements(c, seed)).deposit(float(c["ratio"] ** 3)))
    nu = freqs(n)
    W = 1.0
    for x in nu:
        W = W * torch.sinc(x / n) ** 2
    P = L ** 3 * (dk.real ** 2 + dk.imag ** 2) / (float(n) ** 6 * W * W)
    del dk, W
    r = (nu[0] ** 2 + nu[1] ** 2 + nu[2] ** 2).sqrt()
    w = torch.where((nu[2] > 0) & (nu[2] < n // 2), 2.0, 1.0).to(F64).expand_as(P)
    b = torch.floor(r + 0.5).long().clamp(max=nbins)
    b[0, 0, 0] = nbins
    out = []
    for val in (r * (2 * math.pi / L) * w, P * w, w):
        s = torch.zeros(nbins + 1, dtype=F64, device=DEV)
        for j in range(n):
            s += torch.bincount(b[j].reshape(-1), weights=val[j].reshape(-1), minlength=nbins + 1)
        out.append(s[:nbins])
    k, P, cnt = out
    return {"k": k / cnt.clamp(min=1), "P": P / cnt.clamp(min=1), "n": None}


def exact(case, seed):
    if case["kind"] == "ensemble":
        return [mock_exact(m, s, m["steps"])[0] for m, s in members_of(case, seed)]
    if case["kind"] == "mock":
        u, v = mock_exact(case, seed, case["steps"])
        return {"u": u, "v": v}
    if case["kind"] == "ic":
        return {"u": mock_exact(case, seed, 0)[0]}
    if case["kind"] == "pk":
        return pk_exact(case, seed)
    F, m = pm_exact(case, displacements(case, seed), case["a"], bool(case.get("meshes")))
    out = {"force": F}
    if m:
        out.update(zip(("rho", "src", "fx", "fy", "fz"), m))
    return out
