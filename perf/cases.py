"""The work that a program has this library do, as timed and compared cases.

A case is a dict of plain values.  `prepare` makes what a program has in hand
(device fields made from the seed, a context with its source table, host
catalogues), `run` is one pass through the public entry points, `work` counts
what the pass cannot do without, and `exact` computes the same outputs in plain
torch, in 64 bits, from the method's definitions.

What a case calls ("kind"):
  trace    Context.trace_step: one ray-tracing pass on a resident context
  async    Context.trace_step_async: the same without a host round trip
  noalloc  trace_step_noalloc: the pass of callers that cannot allocate
  rt       Context.set_ionization + rt_step: one radiation step from a given
           ionization (trace and chemistry iterated to convergence)
  density  a coupled step: the density has changed, so a new Context is made
           from it, gets its sources and traces one pass
  merge    clear_sources + add_sources + merge_sources + get_sources: the
           source pre-pass of every radiation step

What the grid holds ("field"):
  uniform    the Stromgren set-up: uniform neutral gas, one source, open box
  lognormal  neutral lognormal gas, uniform sources, mean cell depth tau_cell
  bubbles    cosmological lognormal gas at z = 7, one ionized bubble a source
  clustered  the same gas, sources in clusters of 64, 200 bubbles a 512^3
             volume on cluster centres; the catalogue is merged first
  late       the same gas, 70 % ionized by 5000 overlapping bubbles, sources
             at their centres (the merged catalogue of the late epoch)
"""
import ctypes
import math

import numpy as np
import torch

import paper_2512_12466_amd as nrt

SIGMA0 = 6.30e-18                       # cm^2
KPC_CM = 3.0856775814913673e21
MYR_S = 3.15576e13
ALPHA_B = 2.59e-13                      # cm^3/s at 1e4 K
NH_Z7 = 9.8e-5                          # mean n_H [cm^-3] at z = 7
L_BOX_CM = 40.0 / 0.67742 / 8.0 * 1e3 * KPC_CM   # 40/h comoving Mpc at z = 7
X_IN = 1.0 - 1e-4                       # ionized fraction inside a bubble
N_MIN_RAY, TAU_MAX = 4.0, 30.0
DEV = "cuda:0"


def _case(name, kind, field, n, m, **over):
    c = dict(name=name, kind=kind, field=field, n=n, m=m, precision="mixed", periodic=True,
             l_max=10, capacity=1 << 22, corr=nrt.CORR_CONSERVATIVE, spectrum=nrt.SPEC_MONO,
             spec_param=0.0, tau_cell=0.5)
    c.update(over)
    return c


def listed():
    return [
        # the smallest call: one Stromgren pass, where launches and latency count
        _case("stromgren-32", "trace", "uniform", 32, 1, precision="fp64", periodic=False,
              l_max=7, capacity=1 << 18),
        # one 2 Myr radiation step of the Stromgren test: ~20 small passes and their chemistry
        _case("stromgren-32-step", "rt", "uniform", 32, 1, precision="fp64", periodic=False,
              l_max=7, capacity=1 << 18),
        # an odd, open box with few sources and the default queues
        _case("open-97", "trace", "lognormal", 97, 5, periodic=False, l_max=9),
        # an ordinary neutral box, both precisions, queues as wide as its widest level
        _case("lognormal-128", "trace", "lognormal", 128, 64, l_max=9, capacity=1 << 25),
        _case("lognormal-128-fp64", "trace", "lognormal", 128, 64, precision="fp64", l_max=9,
              capacity=1 << 25),
        # hard photons: every ray lives to the deepest level (long rays, a spectrum table)
        _case("blackbody-128-fp64", "trace", "lognormal", 128, 4, precision="fp64", l_max=9,
              capacity=1 << 25, spectrum=nrt.SPEC_BLACKBODY, spec_param=5e4),
        # a coupled step: new density, new context, one first pass
        _case("density-128", "density", "lognormal", 128, 16, l_max=9),
        # many sources in early bubbles
        _case("bubbles-256", "trace", "bubbles", 256, 4096, capacity=1 << 25),
        # a merged clustered catalogue: very many short rays
        _case("clustered-512", "trace", "clustered", 512, 32768, l_max=11, capacity=1 << 25),
        # the largest grid late in reionization, a few of its sources: long rays in bubbles
        _case("late-1024", "trace", "late", 1024, 96, capacity=1 << 25),
        # the source pre-pass on an ordinary and on the largest catalogue
        _case("merge-512", "merge", "clustered", 512, 32768, l_max=6, capacity=4096),
        _case("merge-1024", "merge", "late", 1024, 262144, l_max=6, capacity=4096),
    ]


def draw(rng):
    def log_int(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    kind = rng.choice(["trace"] * 6 + ["async", "noalloc", "rt", "rt", "density", "merge", "merge"])
    prec = rng.choice(["mixed", "fp64"])
    periodic = rng.random() < 0.7
    if kind == "merge":
        n = log_int(48, 640)
        return _pure(_case("", kind, rng.choice(["clustered", "late"]), n, log_int(64, 200000),
                           l_max=5, capacity=4096, periodic=periodic))
    if kind == "noalloc":
        n = log_int(8, 64)
        return _pure(_case("", kind, "lognormal", n, log_int(1, 8), precision=prec, l_max=6,
                           periodic=periodic, capacity=1 << 17, tau_cell=rng.choice([0.5, 1.0])))
    if kind == "rt":
        # the iteration's count of passes is a whole number: the FP64 path repeats it exactly
        n = log_int(16, 64)
        return _pure(_case("", kind, "uniform" if rng.random() < 0.5 else "lognormal", n,
                           log_int(1, 4), precision="fp64", periodic=periodic, l_max=7,
                           capacity=1 << 20))
    spectrum, param = nrt.SPEC_MONO, 0.0
    field = rng.choice(["lognormal", "lognormal", "bubbles", "clustered", "late"])
    if kind == "trace" and rng.random() < 0.2:
        spectrum, param = rng.choice([(nrt.SPEC_BLACKBODY, 5e4), (nrt.SPEC_BLACKBODY, 3e4),
                                      (nrt.SPEC_POWERLAW, 4.0)])
    n = log_int(12, 128 if spectrum else 384)
    l_max = 11 if n > 160 else (10 if n > 80 else 9)
    cap = 1 << rng.choice([20, 22, 25])
    if kind == "async":  # the pass that cannot fall back: queues that hold its widest level
        n, l_max, cap = log_int(12, 96), 8, 1 << 24
    most = {"lognormal": 64, "bubbles": 4096, "clustered": 16384, "late": 96}[field]
    if spectrum or kind == "async":
        most = 4
    return _pure(_case("", kind, field, n, log_int(1, most), precision=prec, periodic=periodic,
                       l_max=l_max, capacity=cap, corr=rng.choice([2, 2, 2, 0, 1, 3, 4]),
                       spectrum=spectrum, spec_param=param, tau_cell=rng.choice([0.3, 0.5, 1.0])))


def _pure(case):
    case.pop("name")
    return case


# ---- inputs -----------------------------------------------------------------

def _gen(seed, stream):
    g = torch.Generator(device=DEV)
    g.manual_seed(12466 + 1000003 * int(seed) + stream)
    return g


def _normal(shape, g):
    return torch.randn(shape, dtype=torch.float64, device=DEV, generator=g)


def _uniform(shape, g):
    return torch.rand(shape, dtype=torch.float64, device=DEV, generator=g)


def _lognormal_gas(n, mean, sigma, g):
    """mean * exp(sigma g - sigma^2/2), g a unit Gaussian field with P(k) ~ k^-2."""
    f = _normal((n, n, n), g)
    fk = torch.fft.rfftn(f)
    del f
    k = torch.fft.fftfreq(n, device=DEV, dtype=torch.float64) * n
    kz = torch.arange(n // 2 + 1, device=DEV, dtype=torch.float64)
    for a in range(0, n, 64):
        k2 = (k[a:a + 64, None, None] ** 2 + k[None, :, None] ** 2 + kz[None, None, :] ** 2)
        fk[a:a + 64] *= torch.where(k2 > 0, k2.clamp_min(1.0).rsqrt(), 0.0)
    f = torch.fft.irfftn(fk, s=(n, n, n))
    del fk
    f -= f.mean()
    f *= sigma / (f.square().mean().sqrt() + 1e-300)
    return f.sub_(0.5 * sigma ** 2).exp_().mul_(mean)


def _rates(m, sigma, g):
    return 1e50 * torch.exp(sigma * _normal((m,), g) - 0.5 * sigma ** 2)


def _positions(m, n, g):
    return torch.minimum(_uniform((m, 3), g) * n,
                         torch.tensor(np.nextafter(float(n), 0.0), device=DEV).double())


def _paint(x, n, centres, radii, periodic):
    """x_in in every cell whose centre lies within a bubble (centres in x, y, z order)."""
    flat = x.view(-1)
    size = torch.ceil(radii).long() + 1
    for half in size.unique().tolist():
        sel = (size == half).nonzero().view(-1)
        o = torch.arange(-half, half + 1, device=DEV)
        chunk = max(1, (1 << 25) // o.numel() ** 3)
        for b in range(0, sel.numel(), chunk):
            c, r = centres[sel[b:b + chunk]], radii[sel[b:b + chunk]]
            i = torch.floor(c).long()[:, :, None] + o                        # (b, 3, w)
            d2 = (i + 0.5 - c[:, :, None]).square()
            inside = (d2[:, 2, :, None, None] + d2[:, 1, None, :, None]
                      + d2[:, 0, None, None, :]) <= r.square()[:, None, None, None]
            w = i % n if periodic else i.clamp(0, n - 1)
            idx = w[:, 0, None, None, :] + n * (w[:, 1, None, :, None] + n * w[:, 2, :, None, None])
            flat[idx[inside]] = X_IN
    return x


def _inputs(case, seed):
    """Device fields n_H and x, and the host catalogue (pos, ndot)."""
    n, m, field, periodic = case["n"], case["m"], case["field"], case["periodic"]
    g = _gen(seed, 1)
    if field == "uniform":
        # the density and the source vary a little with the seed
        u = _uniform((5,), g).cpu().numpy()
        n_H = torch.full((n, n, n), 1e-3 * (0.9 + 0.2 * u[0]), dtype=torch.float64, device=DEV)
        x = torch.zeros_like(n_H)
        pos = _positions(m, n, g) if m > 1 else torch.tensor(
            [n / 2 + 0.5 + 0.2 * (u[1:4] - 0.5)], device=DEV)
        return n_H, x, 6.6 * KPC_CM / n, pos.cpu().numpy(), 5e48 * (0.9 + 0.2 * u[4]) * np.ones(m)
    if field == "lognormal":
        n_H = _lognormal_gas(n, 1e-3, 1.0, g)
        x = torch.zeros_like(n_H)
        h = case["tau_cell"] / (SIGMA0 * 1e-3)
        pos, ndot = _positions(m, n, g), _rates(m, 1.0, g)
        return n_H, x, h, pos.cpu().numpy(), ndot.cpu().numpy()
    n_H = _lognormal_gas(n, NH_Z7, 1.5, g)
    x = torch.zeros_like(n_H)
    h = L_BOX_CM / n
    if field == "bubbles":
        pos, ndot = _positions(m, n, g), _rates(m, 2.0, g)
        r = (6.0 * (ndot / 1e50) ** (1 / 3)).clamp(2.0, 32.0) * (n / 256)
        _paint(x, n, pos, r, periodic)
        return n_H, x, h, pos.cpu().numpy(), ndot.cpu().numpy()
    if field == "late" and case["kind"] != "merge":
        # the merged catalogue: one source a cluster, its rate the sum of 64 members
        nb = 5000
        centres = _uniform((nb, 3), g) * n
        r = 36.6 * (n / 1024) * (0.5 + _uniform((nb,), g))
        _paint(x, n, centres, r, periodic)
        pos = torch.floor(centres[:m]).clamp(0, n - 1) + 0.5
        ndot = _rates(64 * m, 2.0, g).view(m, 64).sum(1)
        return n_H, x, h, pos.cpu().numpy(), ndot.cpu().numpy()
    # clusters of 64 cell-snapped sources, 2 cells wide
    k = -(-m // 64)
    centres = _uniform((k, 3), g) * n
    pos = (centres[:, None, :] + 2.0 * _normal((k, 64, 3), g)).view(-1, 3)[:m]
    pos = torch.floor(pos).long() % n + 0.5
    ndot = _rates(m, 2.0, g)
    if field == "clustered":
        nb = max(1, min(k, int(200 * (n / 512) ** 3)))
        _paint(x, n, centres[:nb], 4.0 + 16.0 * _uniform((nb,), g), periodic)
    else:
        nb = 5000
        more = _uniform((max(0, nb - k), 3), g) * n
        centres = torch.cat([centres, more])[:nb]
        _paint(x, n, centres, 36.6 * (n / 1024) * (0.5 + _uniform((nb,), g)), periodic)
    return n_H, x, h, pos.cpu().numpy(), ndot.cpu().numpy()


def _desc(case, h):
    n_th = 1e-5 if case["field"] in ("uniform", "lognormal") else 1e-2 * NH_Z7
    return nrt.make_desc(case["n"], h, periodic=case["periodic"], sigma0=SIGMA0,
                         n_min_ray=N_MIN_RAY, l_max=case["l_max"], tau_max=TAU_MAX, n_th=n_th,
                         corr=case["corr"], spectrum=case["spectrum"],
                         spec_param=case["spec_param"],
                         precision=nrt.MIXED if case["precision"] == "mixed" else nrt.FP64)


def _traced_sources(case, n_H, x, h, pos, ndot):
    """The catalogue that is traced: the clustered one is merged first."""
    if case["field"] != "clustered":
        return pos, ndot
    ctx = nrt.Context(nrt.make_desc(case["n"], h, periodic=case["periodic"], l_max=0), n_H, x,
                      max_sources=len(ndot), ray_capacity=4096, device=DEV)
    ctx.add_sources(pos, ndot)
    ctx.merge_sources()
    pos, ndot, _ = ctx.get_sources()
    ctx.destroy()
    return pos, ndot


def prepare(case, seed):
    n_H, x, h, pos, ndot = _inputs(case, seed)
    kind, desc = case["kind"], _desc(case, h)
    s = dict(kind=kind, desc=desc, capacity=case["capacity"])
    if kind == "merge":
        s["pos"], s["ndot"] = pos, ndot
        s["out"] = [np.zeros_like(pos), np.zeros_like(ndot), np.zeros_like(ndot)]
    else:
        pos, ndot = _traced_sources(case, n_H, x, h, pos, ndot)
        s["gamma"] = torch.empty_like(n_H)
    if kind in ("density", "noalloc"):
        s.update(n_H=n_H, x=x, pos=pos, ndot=ndot)
        return s
    s["ctx"] = nrt.Context(desc, n_H, x, max_sources=max(len(ndot), 1),
                           ray_capacity=case["capacity"], device=DEV)
    if kind == "rt":
        s["x"] = x
    if kind == "async":
        s["budget"] = torch.empty(nrt.C.sizeof(nrt.Budget), dtype=torch.uint8, device=DEV)
        s["dropped"] = torch.empty(1, dtype=torch.int64, device=DEV)
    if kind != "merge":
        s["ctx"].add_sources(pos, ndot)
    return s


# ---- one pass ---------------------------------------------------------------

def run(s):
    kind = s["kind"]
    if kind == "trace":
        return s["ctx"].trace_step(s["gamma"])
    if kind == "async":
        gamma, b, dropped = s["ctx"].trace_step_async(s["gamma"], s["budget"], s["dropped"])
        return gamma, b.view(torch.float64)[:4], b.view(torch.int64)[4:], dropped
    if kind == "noalloc":
        b = nrt.trace_step_noalloc(s["desc"], s["n_H"], s["x"], s["pos"], s["ndot"], s["gamma"],
                                   s["capacity"])
        return s["gamma"], b
    if kind == "rt":
        s["ctx"].set_ionization(s["x"])
        gamma, b, passes = s["ctx"].rt_step(2.0 * MYR_S, ALPHA_B, gamma=s["gamma"],
                                            conv_frac=1e-3, max_iter=60)
        return gamma, b, passes, s["ctx"].get_ionization()
    if kind == "density":
        ctx = nrt.Context(s["desc"], s["n_H"], s["x"], max_sources=len(s["ndot"]),
                          ray_capacity=s["capacity"], device=DEV)
        ctx.add_sources(s["pos"], s["ndot"])
        gamma, b = ctx.trace_step(s["gamma"])
        ctx.destroy()
        return gamma, b
    ctx = s["ctx"]
    ctx.clear_sources()
    ctx.add_sources(s["pos"], s["ndot"])
    k = ctx.merge_sources()
    # the catalogue goes into the program's arrays, which hold the largest one
    for out, got in zip(s["out"], ctx.get_sources()):
        out[:k] = got
    return k, s["out"]


# ---- what a pass cannot do without ------------------------------------------

def _segments(case):
    """Cell segments of a pass, estimated: a source's rays by level, to where
    the gas has absorbed them or the box ends."""
    n = case["n"]
    end = math.sqrt(3.0) * n if case["periodic"] else 0.55 * n
    if case["spectrum"] == nrt.SPEC_MONO:
        if case["field"] == "lognormal":
            end = min(end, 1.1 * TAU_MAX / case["tau_cell"])
        elif case["field"] == "bubbles":
            end = min(end, 0.06 * n)
        elif case["field"] == "clustered":
            end = min(end, 0.013 * n)
        elif case["field"] == "late":
            end = min(end, 0.16 * n)
    segs, r0 = 0.0, 0.0
    for level in range(case["l_max"] + 1):
        r1 = math.sqrt(12 * 4 ** level / (N_MIN_RAY * 4 * math.pi))
        segs += 1.5 * 12 * 4 ** level * max(0.0, min(r1, end) - r0)
        r0 = r1
    m = case["m"] if case["field"] != "clustered" else 0.6 * case["m"]
    return m * segs


def work(case):
    cells, m = case["n"] ** 3, case["m"]
    if case["kind"] == "merge":
        # the catalogue in and out, the shells' samples once, about 20 operations each
        samples = m * 4 * 500
        return {"bytes": 32 * m + 40 * m + min(8 * cells, 8 * samples), "flops": 20.0 * samples}
    fields = 32 if case["kind"] == "rt" else (24 if case["kind"] in ("density", "noalloc") else 16)
    passes = 8 if case["kind"] == "rt" else 1
    return {"bytes": float(fields * cells + 32 * m),
            "flops": passes * 70.0 * max(_segments(case), 1.0)}


# ---- the same outputs in plain torch, 64 bits -------------------------------

class _Directions:
    """HEALPix nested pixel centres (Gorski et al. 2005)."""
    top = -1

    def _angles(self, level):
        """The C library's joint cosine and sine of pi k / (4 nr), 1 <= k < nr <= 2^level
        (an ulp off turns face choices at near ties, which Gamma shows)."""
        self.top = level
        shape = ((1 << level) + 1,) * 2
        nr, k = np.tril_indices(shape[0], -1)
        nr, k = nr[k > 0], k[k > 0]
        ang = ((math.pi * k) / (4 * nr)).tolist()
        c, s = np.zeros(shape), np.zeros(shape)
        sincos, arg = ctypes.CDLL("libm.so.6").sincos, ctypes.c_double
        sincos.argtypes, sincos.restype = [arg, ctypes.c_void_p, ctypes.c_void_p], None
        sc = np.empty((len(ang), 2))
        at = sc.ctypes.data
        for q, a in enumerate(ang):
            sincos(a, at + 16 * q, at + 16 * q + 8)
        s[nr, k], c[nr, k] = sc[:, 0], sc[:, 1]
        self.cos, self.sin = (torch.tensor(v, device=DEV) for v in (c, s))

    def _rings(self, ns):
        """Pixels a quarter, height and its sine, by ring."""
        jr = np.arange(4 * ns + 1)
        nr = np.minimum(np.minimum(jr, 4 * ns - jr), ns)
        t = (nr * nr) / float(3 * ns * ns)
        zb = (4 * ns - 2 * jr) / float(3 * ns)
        z = np.where(jr < ns, 1.0 - t, np.where(jr > 3 * ns, t - 1.0, zb))
        st = np.sqrt(np.where((jr < ns) | (jr > 3 * ns), t * (2.0 - t),
                              (1.0 - np.clip(zb, -1, 1)) * (1.0 + np.clip(zb, -1, 1))))
        return (torch.tensor(v, device=DEV) for v in (nr, z, st))

    def __call__(self, level, pix):
        if level > self.top:
            self._angles(max(6, level))
        ns = 1 << level
        face = pix >> (2 * level)
        ipf = pix & ((1 << (2 * level)) - 1)
        ix, iy = torch.zeros_like(pix), torch.zeros_like(pix)
        for b in range(level):
            ix |= ((ipf >> (2 * b)) & 1) << b
            iy |= ((ipf >> (2 * b + 1)) & 1) << b
        row = face >> 2
        jr = (row + 2) * ns - ix - iy - 1
        nr, z, st = (v[jr] for v in self._rings(ns))
        num = (2 * (face & 3) + (row != 1).long()) * nr + ix - iy
        num = torch.where(num < 0, num + 8 * nr, num)
        num = torch.where(num >= 8 * nr, num - 8 * nr, num)
        quad = (num >= 2 * nr).long() + (num >= 4 * nr).long() + (num >= 6 * nr).long()
        rem = num - quad * 2 * nr
        low = rem < nr
        k = torch.where(low, rem, 2 * nr - rem)
        kk = torch.where((rem == 0) | (rem == nr), 1, k).clamp_max(self.cos.shape[0] - 1)
        ca, sa = self.cos[nr, kk], self.sin[nr, kk]
        c, s = torch.where(low, ca, sa), torch.where(low, sa, ca)
        half = math.sqrt(0.5)
        c = torch.where(rem == 0, 1.0, torch.where(rem == nr, half, c))
        s = torch.where(rem == 0, 0.0, torch.where(rem == nr, half, s))
        cx = torch.where(quad == 0, c, torch.where(quad == 1, -s, torch.where(quad == 2, -c, s)))
        sy = torch.where(quad == 0, s, torch.where(quad == 1, c, torch.where(quad == 2, -s, -c)))
        return torch.stack([st * cx, st * sy, z], 1)


class _Mono:
    chunk = 1 << 21

    def at(self, tau):                          # what the other functions need of tau
        return torch.exp(-tau)

    def share(self, e):                         # photons left
        return e

    def taken(self, e, dtau):                   # photons absorbed across dtau
        return e * -torch.expm1(-dtau)

    def thin(self, e):                          # the same per dtau, for dtau -> 0
        return e

    def stopped(self, tau, e):
        return tau >= TAU_MAX


class _Spectrum:
    """Frequency integrals by composite Gauss-Legendre quadrature: over nu/nu_0
    for a blackbody, over (nu/nu_0)^-3 for a power law."""
    chunk = 1 << 18

    def __init__(self, kind, param):
        x, w = np.polynomial.legendre.leggauss(20)
        if kind == nrt.SPEC_BLACKBODY:
            beta = 13.6 / 8.617333262e-5 / param
            edges = 1.0 + np.array([0.0, 0.7, 3.0, 9.0, 20.0, 45.0]) / beta
        else:
            edges = np.array([0.0, 1e-2, 0.1, 0.4, 1.0])
        mid, half = 0.5 * (edges[1:] + edges[:-1]), 0.5 * (edges[1:] - edges[:-1])
        u = (mid[:, None] + half[:, None] * x).ravel()
        w = (half[:, None] * w).ravel()
        if kind == nrt.SPEC_BLACKBODY:
            w, s = w * u * u / np.expm1(beta * u), u ** -3.0
        else:
            w, s = w * u ** ((param - 4.0) / 3.0), u
        self.s, self.w = (torch.tensor(v, device=DEV) for v in (s, w / w.sum()))

    def at(self, tau):
        return torch.exp(tau[:, None] * -self.s)

    def share(self, e):
        return e @ self.w

    def taken(self, e, dtau):
        return (torch.expm1(dtau[:, None] * -self.s) * e) @ -self.w

    def thin(self, e):
        return e @ (self.w * self.s)

    def stopped(self, tau, e):
        return self.share(e) <= math.exp(-TAU_MAX)


def _plane(o, d, i):
    t = ((torch.where(d > 0, i + 1, i)).double() - o) / d
    return torch.where(d != 0, t, math.inf)


def _march(case, desc, absorber, n_H, pos, l0, spec, dirs, level, src, pix, s, tau, gamma, tot):
    """Marches rays of one level to their end; returns those that split."""
    n, h, per, corr = case["n"], desc.h_cm, case["periodic"], case["corr"]
    omega = 4 * math.pi / (12 * 4.0 ** level)
    r2 = 1.0 / (N_MIN_RAY * omega)
    s_max = math.sqrt(3.0) * n if per else math.inf
    rate = l0[src] * 4.0 ** -level
    o, d = pos[src], dirs(level, pix)
    q = o + s[:, None] * d
    f = torch.floor(q)
    i = f.long() - ((q == f) & (d < 0)).long()
    t = _plane(o, d, i)
    step = d.sign().long()
    ids = torch.stack([src, pix], 1)
    split = []

    def book(name, mask, photons):
        tot[name] += float(photons[mask].sum())

    def keep(mask):
        nonlocal o, d, i, t, s, tau, rate, step, ids
        o, d, i, t, s, tau, rate, step, ids = (v[mask] for v in (o, d, i, t, s, tau, rate, step,
                                                                  ids))

    def outside():
        return ((i < 0) | (i >= n)).any(1)

    if not per:
        out = outside()
        book("escaped", out, rate * spec.share(spec.at(tau)))
        keep(~out)
    stride = torch.tensor([1, n, n * n], device=DEV)
    while s.numel():
        far = s >= s_max
        e = spec.at(tau)
        deep = ~far & spec.stopped(tau, e)
        due = ~far & ~deep & (s * s > r2)
        end = far | deep | due
        if bool(end.any()):
            left = rate * spec.share(e)
            book("escaped", far, left)
            book("truncated", deep, left)
            if level >= case["l_max"]:
                book("truncated", due, left)
            else:
                split.append((ids[due], s[due], tau[due]))
            e = e[~end]
            keep(~end)
            if not s.numel():
                break
        tn, ax = t.min(1)
        ax = torch.where(t[:, 0] == tn, 0, torch.where(t[:, 1] == tn, 1, 2))
        ds = (tn - s).clamp_min(0.0)
        c = ((i % n) * stride).sum(1)
        a = absorber[c]
        dl = ds * h
        dtau = SIGMA0 * a * dl
        took = rate * spec.taken(e, dtau)
        G = took / (a * h ** 3)
        thin = a == 0
        if bool(thin.any()):
            G = torch.where(thin, rate * spec.thin(e) * SIGMA0 * dl / h ** 3, G)
        tot["absorbed"] += float(took.sum())
        fc = torch.ones_like(ds)
        if corr != nrt.CORR_NONE:
            rm = 0.5 * (s + tn)
            lpix = rm * math.sqrt(omega)
            mid = o + rm[:, None] * d
            dm, dp = mid - i.double(), (i + 1).double() - mid
            side = torch.where(dm < dp, -1, torch.where(dp < dm, 1, torch.where(d < 0, -1, 1)))
            da = torch.where(dm < dp, dm, dp)
            edge = da.min(1).values
            fax = torch.where(da[:, 0] == edge, 0, torch.where(da[:, 1] == edge, 1, 2))
            j = i.clone()
            j.scatter_add_(1, fax[:, None], side.gather(1, fax[:, None]))
            c2 = ((j % n) * stride).sum(1)
            usable = (n_H[c2] >= desc.n_th) & (absorber[c2] > 0)
            if not per:
                usable &= ((j >= 0) & (j < n)).all(1)
            near = edge < 0.5 * lpix
            lin = 0.5 + edge / lpix
            if corr == nrt.CORR_CONSERVATIVE:
                fc = torch.where(near & usable, lin, 1.0)
            elif corr == nrt.CORR_SQUARED:
                fc = torch.where(near, lin * lin, 1.0)
            else:
                fc = torch.where(near, lin, 1.0)
            if corr in (nrt.CORR_CONSERVATIVE, nrt.CORR_NAIVE):
                u = usable
                gamma.index_add_(0, c2[u], ((1.0 - fc) * (a / absorber[c2]) * G)[u])
        gamma.index_add_(0, c, fc * G)
        tau = tau + dtau
        s = tn
        i.scatter_add_(1, ax[:, None], step.gather(1, ax[:, None]))
        t = _plane(o, d, i)
        tot["segments"] += int(s.numel())
        if not per:
            out = outside()
            if bool(out.any()):
                book("escaped", out, rate * spec.share(spec.at(tau)))
                keep(~out)
    return split


def _exact_pass(case, desc, n_H, x, pos, ndot, dirs):
    n = case["n"]
    absorber = ((1.0 - x) * n_H).view(-1)
    flat_n = n_H.view(-1)
    gamma = torch.zeros(n ** 3, dtype=torch.float64, device=DEV)
    spec = (_Mono() if case["spectrum"] == nrt.SPEC_MONO
            else _Spectrum(case["spectrum"], case["spec_param"]))
    P = torch.tensor(np.asarray(pos), dtype=torch.float64, device=DEV).view(-1, 3)
    L = torch.tensor(np.asarray(ndot), dtype=torch.float64, device=DEV) / 12.0
    m = L.numel()
    tot = dict(emitted=float(sum(np.asarray(ndot).tolist())), absorbed=0.0, escaped=0.0,
               truncated=0.0, segments=0, rays=0, splits=0, rays_per_level=[0] * 15)
    src = torch.arange(m, device=DEV).repeat_interleave(12)
    pix = torch.arange(12, device=DEV).repeat(m)
    s = torch.zeros(12 * m, dtype=torch.float64, device=DEV)
    tau = s.clone()
    for level in range(case["l_max"] + 1):
        tot["rays"] += int(s.numel())
        tot["rays_per_level"][level] = int(s.numel())
        split = []
        for b in range(0, s.numel(), spec.chunk):
            e = slice(b, b + spec.chunk)
            split += _march(case, desc, absorber, flat_n, P, L, spec, dirs, level, src[e], pix[e],
                            s[e], tau[e], gamma, tot)
        if not split:
            break
        ids, s, tau = (torch.cat([v[k] for v in split]) for k in range(3))
        tot["splits"] += int(s.numel())
        src = ids[:, 0].repeat_interleave(4)
        pix = (4 * ids[:, 1:2] + torch.arange(4, device=DEV)).view(-1)
        s, tau = s.repeat_interleave(4), tau.repeat_interleave(4)
        if not s.numel():
            break
    return gamma.view(n, n, n), tot


def _exact_chem(G, n_H, x0, dt, alpha, guess):
    xav, xn = guess.clone(), x0.clone()
    live = torch.ones_like(xav, dtype=torch.bool)
    for _ in range(200):
        rate = G + (xav * n_H) * alpha
        ti = 1.0 / rate
        xeq = G * ti
        u = dt / ti
        mean = torch.where(rate > 0, xeq + (x0 - xeq) * (-torch.expm1(-u) / u), x0)
        end = torch.where(rate > 0, xeq + (x0 - xeq) * torch.exp(-u), x0)
        moved = (mean - xav).abs() > 1e-12
        xav, xn = torch.where(live, mean, xav), torch.where(live, end, xn)
        live &= moved
        if not bool(live.any()):
            break
    return xn, xav


def _exact_merge(case, x, pos, ndot):
    n, per = case["n"], case["periodic"]
    # the parameters that merge_sources takes by default
    dr, x_th, f_req, n_min, r_max, f_ov, eps = 2.0, 0.9, 0.9, 8, 8.0, 1.0, 1e-6
    cell = torch.floor(torch.tensor(pos, device=DEV)).long()
    key = (cell[:, 0] * n + cell[:, 1]) * n + cell[:, 2]
    uniq, inv = torch.unique(key, return_inverse=True)
    flux = torch.zeros(uniq.numel(), dtype=torch.float64, device=DEV)
    flux.index_add_(0, inv, torch.tensor(ndot, device=DEV))
    cell = torch.stack([uniq // (n * n), (uniq // n) % n, uniq % n], 1)
    m = uniq.numel()
    stride = torch.tensor([1, n, n * n], device=DEV)
    xf = x.view(-1)
    d = _Directions()(3, torch.arange(768, device=DEV))
    radius = torch.zeros(m, dtype=torch.float64, device=DEV)
    live = xf[(cell * stride).sum(1)] >= x_th
    for k in range(1, int(r_max / dr) + 1):
        who = live.nonzero().view(-1)
        for b in range(0, who.numel(), 1 << 14):
            w = who[b:b + (1 << 14)]
            v = torch.floor((cell[w] + 0.5)[:, None, :] + k * dr * d).long()
            ok = torch.ones(v.shape[:2], dtype=torch.bool, device=DEV)
            if not per:
                ok = ((v >= 0) & (v < n)).all(2)
            c = torch.where(ok, ((v % n) * stride).sum(2), -1).sort(1).values
            first = (c >= 0) & torch.cat([torch.ones_like(c[:, :1], dtype=torch.bool),
                                          c[:, 1:] != c[:, :-1]], 1)
            tot = first.sum(1)
            ion = (first & (xf[c.clamp_min(0)] >= x_th)).sum(1)
            good = torch.where(tot < n_min, ion == tot,
                               ~(ion.double() / tot.double() < f_req))
            radius[w[good]] = k * dr
            live[w[~good]] = False
    radius[live] = r_max
    has = (radius > 0).nonzero().view(-1)

    def image(v):
        if not per:
            return v
        v = v % n
        return torch.where(2 * v > n, v - n, v)

    label = torch.arange(m, device=DEV)
    ea, eb = [], []
    for b in range(0, has.numel(), 256):
        w, rest = has[b:b + 256], has[b:]
        d2 = image(cell[w][:, None, :] - cell[rest][None]).double().square().sum(2)
        near = d2 <= (f_ov * (radius[w][:, None] + radius[rest][None])).square() + eps
        p = near.nonzero()
        p = p[p[:, 0] < p[:, 1]]
        ea.append(w[p[:, 0]])
        eb.append(rest[p[:, 1]])
    if ea:
        ea, eb = torch.cat(ea), torch.cat(eb)
        while True:
            low = torch.minimum(label[ea], label[eb])
            new = label.scatter_reduce(0, ea, low, "amin").scatter_reduce(0, eb, low, "amin")
            new = new[new]
            if bool((new == label).all()):
                break
            label = new
    root, group = torch.unique(label, return_inverse=True)
    g = root.numel()
    fsum = torch.zeros(g, dtype=torch.float64, device=DEV).index_add_(0, group, flux)
    rad = torch.zeros(g, dtype=torch.float64, device=DEV).scatter_reduce(0, group, radius, "amax")
    lead = cell[label]
    un = (lead + image(cell - lead)).double()
    cen = torch.zeros((g, 3), dtype=torch.float64, device=DEV).index_add_(
        0, group, flux[:, None] * un) / fsum[:, None]
    rnd = torch.floor(cen + 0.5).long()
    if per:
        rnd = rnd % n
    d2 = image(cell - rnd[group]).square().sum(1)
    rank = d2 * (1 << 20) + torch.arange(m, device=DEV)
    best = torch.full((g,), 1 << 62, dtype=torch.long, device=DEV).scatter_reduce(
        0, group, rank, "amin") % (1 << 20)
    alone = torch.bincount(group, minlength=g) == 1
    out = torch.where(alone[:, None], cell[root], cell[best])
    order = ((out[:, 0] * n + out[:, 1]) * n + out[:, 2]).argsort()
    return [v[order].cpu().numpy() for v in (out.double() + 0.5, fsum, rad)]


def exact(case, seed):
    cost = _segments(case) * (30 if case["spectrum"] else 1)
    if case["kind"] != "merge" and cost > 1.2e10:
        return None  # over 20 seconds
    if case["kind"] == "merge" and case["m"] > 1 << 17:
        return None
    n_H, x, h, pos, ndot = _inputs(case, seed)
    if case["kind"] == "merge":
        got = _exact_merge(case, x, pos, ndot)
        out = [np.zeros_like(pos), np.zeros_like(ndot), np.zeros_like(ndot)]
        for o, v in zip(out, got):
            o[:len(v)] = v
        return len(got[1]), out
    desc = _desc(case, h)
    if case["field"] == "clustered":
        pos, ndot, _ = _exact_merge(case, x, pos, ndot)
    dirs = _Directions()
    if case["kind"] == "rt":
        xav = x.clone()
        for it in range(1, 61):
            gamma, b = _exact_pass(case, desc, n_H, xav, pos, ndot, dirs)
            xn, new = _exact_chem(gamma, n_H, x, 2.0 * MYR_S, ALPHA_B, xav)
            moved = int(((new - xav).abs() >= 1e-6).sum())
            xav = new
            if moved <= math.floor(1e-3 * n_H.numel()):
                break
        return gamma, b, it, xn
    gamma, b = _exact_pass(case, desc, n_H, x, pos, ndot, dirs)
    if case["kind"] == "async":
        parts = [b[k] for k in ("emitted", "absorbed", "escaped", "truncated")]
        return (gamma, torch.tensor(parts, dtype=torch.float64, device=DEV),
                torch.tensor([b["segments"], b["rays"], b["splits"]] + b["rays_per_level"],
                             device=DEV), torch.zeros(1, dtype=torch.int64, device=DEV))
    return gamma, b
