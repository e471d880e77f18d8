"""The work that users of this package have it do, as measurable cases.

A case is a dict of plain values.  `prepare` makes what a program holds before
the call (a lattice with its state, inputs on the device), `run` is one pass
through the public entry points, `work` the bytes and operations the pass
cannot do without, and `exact` the same outputs from plain torch in 64 bits.

Models, box sizes and time steps are those of paper_0911_5692_amd/workloads.py:
  lphi4:  lambda phi^4 + g^2 phi^2 chi^2 / 2 (r = 1, s = -1), white noise of
          1e-3 around f1 = 1, L = 20, dt = dx/20;
  m2phi2: m^2 phi^2 / 2 + g^2 phi^2 chi^2 / 2 (r = 3/2, s = 0), vacuum
          fluctuations around f1 = 1, dx = 10/512, dt = 2^-10.
"""
import math

import numpy as np
import torch

from paper_0911_5692_amd import Ensemble, Lattice, LeapfrogLoss, vacuum_fields
from paper_0911_5692_amd import workloads as W

DEV = "cuda"
DTYPES = {"f32": torch.float32, "f64": torch.float64}
# program-unit a'(0) of f1 = 1, f2 = 0 at rest in the lphi4 model (V = 1/4)
AD0_LPHI4 = math.sqrt(W.KAPPA2 / 3.0 * 0.25)


# ------------------------------------------------------------------- the cases

def listed():
    return [
        # the smallest configuration of the package, whole: initialise, 200 steps, read the result (FP64)
        dict(name="run_32_f64", kind="run", N=32, dtype="f64", stencil=7, model="lphi4", steps=200),
        # a ragged size with the 27-point Laplacian, between two snapshots of a long run
        dict(name="evolve_100_f32_s27", kind="evolve", N=100, dtype="f32", stencil=27, model="m2phi2", steps=100),
        # a lattice that stays in the caches of the part
        dict(name="evolve_128_f32", kind="evolve", N=128, dtype="f32", stencil=7, model="m2phi2", steps=100),
        # one short run of a scan over initial states in FP64
        dict(name="run_160_f64", kind="run", N=160, dtype="f64", stencil=7, model="lphi4", steps=20),
        # the same at the ordinary size in FP32
        dict(name="run_256_f32", kind="run", N=256, dtype="f32", stencil=7, model="lphi4", steps=50),
        # the configuration the paper times: 27-point Laplacian at 256^3 and, at the end, rho and p
        dict(name="evolve_256_f32_s27", kind="evolve_rho_p", N=256, dtype="f32", stencil=27, model="m2phi2", steps=50),
        # the benchmark's lattice, between two snapshots
        dict(name="evolve_512_f32", kind="evolve", N=512, dtype="f32", stencil=7, model="m2phi2", steps=20),
        # the diagnostics of one output time: energies, and rho and p per site
        dict(name="diagnostics_512_f32", kind="diagnostics", N=512, dtype="f32", stencil=7, model="m2phi2"),
        # the power spectra of the four fields at one output time
        dict(name="spectra_512_f32", kind="spectra", N=512, dtype="f32", stencil=7, model="m2phi2"),
        # the initial state of a run, generated on the device
        dict(name="vacuum_512", kind="vacuum", N=512, model="m2phi2"),
        # a mixed ensemble (sizes of the package's ensemble workload) between two snapshots
        dict(name="ensemble_15_f32", kind="ensemble", sizes="64x11,96x3,160x1", dtype="f32", stencil=7,
             model="lphi4", steps=50),
        # one gradient of a fit: loss after n steps and its gradient (forward and backward)
        dict(name="gradient_128_f32", kind="gradient", N=128, dtype="f32", stencil=7, model="lphi4", steps=100, K=25),
    ]


def _size(rng, lo, hi):
    """A size between lo and hi, spread over its logarithm; odd ones among them."""
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["evolve", "evolve", "evolve_rho_p", "run", "run", "diagnostics", "spectra", "vacuum",
                       "ensemble", "gradient"])
    c = dict(kind=kind, model=rng.choice(["lphi4", "m2phi2"]))
    if kind == "vacuum":
        c.update(N=_size(rng, 32, 400))
        return c
    c.update(dtype=rng.choice(["f32", "f32", "f64"]), stencil=rng.choice([7, 7, 27]))
    if kind in ("evolve", "evolve_rho_p", "ensemble"):
        c["model"] = "m2phi2"  # each pass goes on from the last one: the model of the package's long runs
    if kind in ("evolve", "evolve_rho_p"):
        c.update(N=_size(rng, 20, 320))
        most = 4e8 / c["N"] ** 3  # no dearer than the largest listed case
        c["steps"] = rng.choice([n for n in (11, 17, 40, 64, 100) if n <= max(most, 11)])
    elif kind == "run":
        c.update(N=_size(rng, 20, 256), steps=rng.choice([5, 20, 33]))
    elif kind == "diagnostics":
        c.update(N=_size(rng, 32, 400))
    elif kind == "spectra":
        c.update(N=_size(rng, 32, 400))
    elif kind == "ensemble":
        n, sizes = rng.randint(2, 4), []
        for _ in range(n):
            sizes.append("%dx%d" % (_size(rng, 24, 112), rng.randint(1, 15 // n)))
        c.update(sizes=",".join(sizes), steps=rng.choice([10, 31, 50]))
    else:
        c.update(N=_size(rng, 16, 112), steps=rng.choice([20, 45, 60]), K=rng.choice([8, 15, 20]))
    return c


# ------------------------------------------------------------------- inputs

def _model(model, N, stencil=7):
    """Lattice arguments of a model at its own dx and dt."""
    if model == "lphi4":
        dx = 20.0 / N  # its box side is 20 at every N
        return dict(N=N, L=20.0, dt=dx / 20.0, beta=4, c1=1.0, G=100.0, r=1.0, s=-1.0, kappa2=W.KAPPA2,
                    stencil=stencil)
    return W.CFG3.resized(N).model() | dict(stencil=stencil)


def _noise(N, gen):
    return torch.randn((N, N, N), generator=gen, device=DEV, dtype=torch.float64)


def _mode2(N):
    """|n|^2 of every mode of rfftn."""
    n0 = torch.fft.fftfreq(N, device=DEV, dtype=torch.float64) * N
    n2 = torch.fft.rfftfreq(N, device=DEV, dtype=torch.float64) * N
    return n0[:, None, None] ** 2 + n0[None, :, None] ** 2 + n2[None, None, :] ** 2


def _filtered(w, L, m2, velocity):
    """White noise w with the vacuum spectrum of workloads.py, cut at N/4."""
    N = w.shape[0]
    n = _mode2(N).sqrt_()
    omega = ((2.0 * math.pi / L * n) ** 2 + m2).sqrt_()
    P = omega * (W.EPS_VACUUM ** 2 / 2.0) if velocity else (W.EPS_VACUUM ** 2 / 2.0) / omega
    P[(n == 0) | (n > N / 4)] = 0.0
    return torch.fft.irfftn(torch.fft.rfftn(w) * (P * (N / L) ** 3).sqrt_(), s=(N, N, N))


def _state(model, N, seed):
    """f1, f2 and the physical velocities u1, u2 of a run's start (FP64)."""
    gen = torch.Generator(device=DEV)
    gen.manual_seed(seed)
    if model == "lphi4":
        f1 = _noise(N, gen).mul_(1e-3).add_(1.0)
        f2 = _noise(N, gen).mul_(1e-3)
        return f1, f2, torch.zeros_like(f1), torch.zeros_like(f1)
    m = _model(model, N)
    out = []
    for vel in (False, True):
        for m2, mean in ((m["c1"], W.U0_INFLATON if vel else 1.0), (m["G"], 0.0)):
            out.append(_filtered(_noise(N, gen), m["L"], m2, vel).add_(mean).contiguous())
    return tuple(out)


def _spec(model, N, seed):
    m = _model(model, N)
    return dict(f0=(1.0, 0.0), u0=(W.U0_INFLATON, 0.0), m2=(m["c1"], m["G"]), eps2=W.EPS_VACUUM ** 2, cutoff=0.0,
                seed=seed)


def _sizes(case):
    out = []
    for part in case["sizes"].split(","):
        n, k = part.split("x")
        out += [int(n)] * int(k)
    return out


def prepare(case, seed):
    kind = case["kind"]
    if kind == "vacuum":
        return dict(kind=kind, N=case["N"], L=_model(case["model"], case["N"])["L"],
                    spec=_spec(case["model"], case["N"], seed))
    dtype = DTYPES[case["dtype"]]
    if kind == "ensemble":
        sizes = _sizes(case)
        ens = Ensemble([_model(case["model"], n, case["stencil"]) for n in sizes], dtype=dtype, device=DEV)
        for r, n in enumerate(sizes):
            ens.init_physical(r, *_state(case["model"], n, seed * 1000 + r))
        return dict(kind=kind, ens=ens, steps=case["steps"])
    m = _model(case["model"], case["N"], case["stencil"])
    f1, f2, u1, u2 = _state(case["model"], case["N"], seed)
    if kind == "gradient":
        spec = {k: m[k] for k in ("N", "L", "dt", "beta", "c1", "r", "s", "kappa2", "stencil")}
        spec.update(dtype=dtype, n=case["steps"], K=case["K"], a0=1.0, ad0=AD0_LPHI4)
        v = [u + m["r"] * AD0_LPHI4 * f for u, f in ((u1, f1), (u2, f2))]
        args = [torch.tensor(m["G"], dtype=torch.float64)] + [f1, f2] + v
        return dict(kind=kind, args=[a.requires_grad_() for a in args], spec=spec)
    lat = Lattice(**m, dtype=dtype, device=DEV)
    if kind == "run":
        return dict(kind=kind, lat=lat, fields=(f1, f2, u1, u2), steps=case["steps"])
    lat.init_physical(f1, f2, u1, u2)
    return dict(kind=kind, lat=lat, steps=case.get("steps", 0))


# ------------------------------------------------------------------- one pass

_ROW = ("a", "ad", "hubble", "K1", "K2", "G1", "G2", "P", "rho", "R")


def _row(e):
    """One line of a run's log."""
    return np.array([e[k] for k in _ROW])


def run(state):
    kind = state["kind"]
    if kind == "vacuum":
        return vacuum_fields(state["N"], state["L"], state["spec"])
    if kind == "gradient":
        loss = LeapfrogLoss.apply(*state["args"], state["spec"])
        return (loss.detach(), *torch.autograd.grad(loss, state["args"]))
    if kind == "ensemble":
        ens = state["ens"]
        ens.step(state["steps"])
        log = np.stack([_row(e) for e in ens.energies()])
        return [log] + [ens.fields(r, dtype=ens.dtype) for r in range(ens.R)]
    lat = state["lat"]
    if kind == "spectra":
        return [lat.spectrum(w) for w in ("f1", "f2", "v1", "v2")]
    if kind == "diagnostics":
        log = _row(lat.energies())
        rho, p, avg = lat.rho_p()
        return log, rho, p, np.array([avg["rho"], avg["p"], avg["w"]])
    if kind == "run":
        lat.init_physical(*state["fields"])
    lat.step(state["steps"])
    if kind == "evolve_rho_p":
        rho, p, avg = lat.rho_p(dtype=lat.dtype)
        return (rho, p, np.array([avg["rho"], avg["p"], avg["w"]]), *lat.fields(dtype=lat.dtype))
    return (_row(lat.energies()), *lat.fields(dtype=lat.dtype))


def work(case):
    kind = case["kind"]
    if kind == "vacuum":
        n3 = case["N"] ** 3
        # four arrays written; per array a forward and an inverse real FFT and 60 operations of the generator a site
        return dict(bytes=32.0 * n3, flops=4.0 * n3 * (5.0 * math.log2(n3) + 60.0))
    es = 8 if case["dtype"] == "f64" else 4
    n3 = sum(n ** 3 for n in _sizes(case)) if kind == "ensemble" else case["N"] ** 3
    # a step reads and writes both fields and velocities; its sums are formed on the way
    step = dict(bytes=8.0 * es * n3, flops=(70.0 if case["stencil"] == 7 else 170.0) * n3)
    if kind == "spectra":
        return dict(bytes=4.0 * 2.0 * es * n3, flops=4.0 * n3 * (2.5 * math.log2(n3) + 8.0))
    if kind == "diagnostics":
        return dict(bytes=(4.0 * es + 16.0) * n3, flops=100.0 * n3)
    if kind == "gradient":
        # forward steps, and reverse steps (FP64 cotangents read and written, the stored fields read) with the
        # recomputed states
        n = case["steps"]
        return dict(bytes=n * (2.0 * step["bytes"] + (64.0 + 2.0 * es) * n3), flops=n * (2.0 * step["flops"] + 150.0 * n3))
    b, f = case["steps"] * step["bytes"], case["steps"] * step["flops"]
    if kind == "run":
        b += 32.0 * n3 + 4.0 * es * n3
    # the snapshot: the four arrays out (and rho and p)
    out = 6.0 if kind == "evolve_rho_p" else 4.0
    return dict(bytes=b + (4.0 + out) * es * n3, flops=f + 50.0 * n3)


# ------------------------------------------------------------------- the same in plain torch, 64 bits

# the 27-point stencil's bonds whose first nonzero of (dz, dy, dx) is +1, by weight
_BONDS27 = [(w, d) for w, ds in (
    (14.0 / 30.0, [(1, 0, 0), (0, 1, 0), (0, 0, 1)]),
    (3.0 / 30.0, [(0, 1, -1), (0, 1, 1), (1, -1, 0), (1, 1, 0), (1, 0, -1), (1, 0, 1)]),
    (1.0 / 30.0, [(1, -1, -1), (1, -1, 1), (1, 1, -1), (1, 1, 1)])) for d in ds]
_BONDS7 = [(1.0, d) for d in ((1, 0, 0), (0, 1, 0), (0, 0, 1))]


class _Plain:
    """The leapfrog of Sec. II.B of arXiv:0911.5692, on full fields in FP64."""

    def __init__(self, m, G=None):
        self.m, self.G = m, m["G"] if G is None else G
        self.dx = m["L"] / m["N"]
        self.p1 = -2.0 * m["s"] + (2.0 - m["beta"]) * m["r"]
        self.p2 = -2.0 * m["s"] - 2.0 * m["r"]
        self.bonds = _BONDS27 if m["stencil"] == 27 else _BONDS7

    def lap(self, f):
        if self.m["stencil"] == 7:
            s = -6.0 * f
            for ax in range(3):
                s = s + torch.roll(f, 1, ax) + torch.roll(f, -1, ax)
            return s / self.dx ** 2

        def two(g, ax):
            return torch.roll(g, 1, ax) + torch.roll(g, -1, ax)

        x, y = two(f, 2), two(f, 1)
        xy = two(x, 1)
        inner = -128.0 * f + 14.0 * (x + y) + 3.0 * xy
        outer = 14.0 * f + 3.0 * (x + y) + xy
        return (inner + two(outer, 0)) / (30.0 * self.dx ** 2)

    def grad2(self, f):
        g = torch.zeros_like(f)
        for w, d in self.bonds:
            g += w * (torch.roll(f, tuple(-k for k in d), (0, 1, 2)) - f) ** 2
        return g / self.dx ** 2

    def V(self, f1, f2, a):
        m = self.m
        return m["c1"] * a ** self.p1 * f1 ** m["beta"] / m["beta"] + 0.5 * self.G * a ** self.p2 * f1 ** 2 * f2 ** 2

    def friedmann(self, f, u, a):
        m = self.m
        rho = sum((0.5 * ui ** 2 + 0.5 * a ** (-2.0 * m["s"] - 2.0) * self.grad2(fi)).mean() for fi, ui in zip(f, u))
        rho = rho + self.V(*f, a).mean()
        return (m["kappa2"] / 3.0 * a ** (2.0 - 2.0 * m["r"]) * rho) ** 0.5

    def start(self, f, v, a, ad):
        """Fields half a step ahead of the velocities."""
        h = 0.5 * self.m["dt"]
        return [f[0] + h * v[0], f[1] + h * v[1], v[0], v[1], a + h * ad, ad]

    def start_physical(self, f1, f2, u1, u2):
        a = torch.ones((), dtype=torch.float64, device=f1.device)
        ad = self.friedmann((f1, f2), (u1, u2), a)
        r = self.m["r"]
        return self.start((f1, f2), (u1 + r * ad * f1, u2 + r * ad * f2), a, ad)

    def step(self, f1, f2, v1, v2, a, w):
        m = self.m
        dt, r, s, k2 = m["dt"], m["r"], m["s"], m["kappa2"]
        l1, l2 = self.lap(f1), self.lap(f2)
        # the gradient energy is the Laplacian's own form -<f Lap f>; the mean drops out of it
        Sg = -((f1 - f1.mean()) * l1).mean() - ((f2 - f2.mean()) * l2).mean()
        SV = self.V(f1, f2, a).mean()
        Fa = k2 * a ** (-2.0 * s - 2.0 * r - 1.0) * (Sg / 3.0 + a ** (2.0 * s + 2.0) * SV)
        c = (-s - 2.0) * dt / (4.0 * a)
        disc = 1.0 - 8.0 * c * w - 4.0 * c * dt * Fa
        u = 2.0 * (c * w * w + w + dt * Fa) / ((1.0 - 2.0 * c * w) + disc ** 0.5)
        adh, add = 0.5 * (w + u), (u - w) / dt
        bc = r * (s - r + 2.0) * (adh / a) ** 2 + r * add / a
        al, cp1, cp2 = a ** (-2.0 * s - 2.0), m["c1"] * a ** self.p1, self.G * a ** self.p2
        v1 = v1 + dt * (al * l1 + bc * f1 - cp1 * f1 ** (m["beta"] - 1) - cp2 * f1 * f2 ** 2)
        v2 = v2 + dt * (al * l2 + bc * f2 - cp2 * f1 ** 2 * f2)
        return [f1 + dt * v1, f2 + dt * v2, v1, v2, a + dt * u, u]

    def evolve(self, st, n):
        for _ in range(n):
            st = self.step(*st)
        return st

    def synced(self, f1, f2, v1, v2, a, w):
        h = 0.5 * self.m["dt"]
        return f1 - h * v1, f2 - h * v2, v1, v2, a - h * w, w

    def parts(self, st):
        """Kinetic, gradient (per field) and potential energy densities at the synchronised time."""
        f1, f2, v1, v2, a, w = self.synced(*st)
        hub, al = w / a, 0.5 * a ** (-2.0 * self.m["s"] - 2.0)
        K = [0.5 * (v - self.m["r"] * hub * f) ** 2 for f, v in ((f1, v1), (f2, v2))]
        return K, [al * self.grad2(f) for f in (f1, f2)], self.V(f1, f2, a), a, w

    def row(self, st):
        K, Gr, V, a, w = self.parts(st)
        e = [float(x.mean()) for x in (*K, *Gr, V)]
        a, w, rho, m = float(a), float(w), sum(e), self.m
        R = m["kappa2"] / 3.0 * a ** (2.0 - 2.0 * m["r"]) * rho / w ** 2 - 1.0
        return np.array([a, w, w / a, *e, rho, R])

    def rho_p(self, st):
        K, Gr, V, _, _ = self.parts(st)
        k, g = K[0] + K[1], Gr[0] + Gr[1]
        rho, p = k + g + V, k - g / 3.0 - V
        m = float(rho.mean()), float(p.mean())
        return rho, p, np.array([*m, m[1] / m[0]])


def _vacuum_exact(case, seed):
    """Philox4x32-10 noise (Salmon et al., SC'11) through the vacuum filter."""
    N, m = case["N"], _model(case["model"], case["N"])
    mask, out = 0xFFFFFFFF, []
    for j in range(4):
        c = [torch.arange(N ** 3, device=DEV), 0, j, 0]  # N^3 < 2^32 here
        c = [x if torch.is_tensor(x) else torch.full_like(c[0], x) for x in c]
        k = [seed & mask, seed >> 32]
        for r in range(10):
            p0, p1 = c[0] * 0xD2511F53, c[2] * 0xCD9E8D57
            c = [((p1 >> 32) & mask) ^ c[1] ^ k[0], p1 & mask, ((p0 >> 32) & mask) ^ c[3] ^ k[1], p0 & mask]
            k = [(k[0] + 0x9E3779B9) & mask, (k[1] + 0xBB67AE85) & mask]
        u = [((c[i] << 21 | c[i + 1] >> 11) + 1).double() * 2.0 ** -53 for i in (0, 2)]
        del c, p0, p1
        w = ((-2.0 * u[0].log()).sqrt() * (2.0 * math.pi * u[1]).cos()).reshape(N, N, N)
        del u
        i, vel = j & 1, j >= 2
        mean = (W.U0_INFLATON if vel else 1.0) if i == 0 else 0.0
        out.append(_filtered(w, m["L"], (m["c1"], m["G"])[i], vel) + mean)
    return tuple(out)


def _spectrum_exact(f, L):
    N = f.shape[0]
    F = torch.fft.rfftn(f - f.mean())
    F[0, 0, 0] = f.sum()
    shell = torch.floor(_mode2(N).sqrt_() + 0.5).long()
    w = torch.full((N // 2 + 1,), 2.0, device=DEV, dtype=torch.float64)
    w[0] = 1.0
    if N % 2 == 0:
        w[-1] = 1.0
    w = w.expand(N, N, N // 2 + 1).reshape(-1)
    nb = int(math.floor(math.sqrt(3.0) * (N // 2) + 0.5)) + 1
    count = torch.zeros(nb, device=DEV, dtype=torch.float64).index_add_(0, shell.reshape(-1), w)
    power = torch.zeros(nb, device=DEV, dtype=torch.float64)
    power.index_add_(0, shell.reshape(-1), (F.real ** 2 + F.imag ** 2).reshape(-1) * w)
    power = torch.where(count > 0, power / count.clamp(min=1.0) * (L ** 3 / N ** 6), power)
    return power.cpu().numpy(), count.cpu().numpy()


def _gradient_exact(case, seed):
    from torch.utils.checkpoint import checkpoint

    state = prepare(case, seed)
    m = _model(case["model"], case["N"], case["stencil"])
    G = state["args"][0].detach().to(DEV).requires_grad_()
    f1, f2, v1, v2 = state["args"][1:]
    a = torch.ones((), dtype=torch.float64, device=DEV)
    ad = torch.full((), AD0_LPHI4, dtype=torch.float64, device=DEV)

    def some(G, n, *st):
        return tuple(_Plain(m, G).evolve(list(st), n))

    st = _Plain(m, G).start((f1, f2), (v1, v2), a, ad)
    left = case["steps"]
    while left > 0:
        st = checkpoint(some, G, min(5, left), *st, use_reentrant=False)
        left -= 5
    P = _Plain(m, G)
    g1, g2, w1, w2, ak, w = P.synced(*st)
    l2 = P.lap(g2)
    loss = 0.5 * ((w2 - m["r"] * (w / ak) * g2) ** 2).mean()
    loss = loss + 0.5 * ak ** (-2.0 * m["s"] - 2.0) * -((g2 - g2.mean()) * l2).mean()
    g = torch.autograd.grad(loss, [G, f1, f2, v1, v2])
    return (loss.detach(), g[0].cpu(), *g[1:])


def exact(case, seed):
    kind = case["kind"]
    if kind == "vacuum":
        return _vacuum_exact(case, seed)
    if kind == "gradient":
        return _gradient_exact(case, seed)
    if kind == "ensemble":
        rows, out = [], []
        for r, n in enumerate(_sizes(case)):
            P = _Plain(_model(case["model"], n, case["stencil"]))
            st = P.evolve(P.start_physical(*_state(case["model"], n, seed * 1000 + r)), case["steps"])
            rows.append(P.row(st))
            out.append(tuple(st[:4]))
        return [np.stack(rows)] + out
    P = _Plain(_model(case["model"], case["N"], case["stencil"]))
    st = P.start_physical(*_state(case["model"], case["N"], seed))
    if kind == "spectra":
        return [_spectrum_exact(f, P.m["L"]) for f in P.synced(*st)[:4]]
    if kind == "diagnostics":
        rho, p, avg = P.rho_p(st)
        return P.row(st), rho, p, avg
    st = P.evolve(st, case["steps"])
    if kind == "evolve_rho_p":
        return (*P.rho_p(st), *st[:4])
    return (P.row(st), *st[:4])
