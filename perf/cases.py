"""The work that a user of this framework has it do, as cases that can be timed.

A case is one call pattern of the public entry points: a lattice (or a batch of
lattices) is built once, with its potential and initial packet on the GPU, and
a pass advances it by a number of steps, as a simulation loop does between two
looks at the state.  `prepare` makes what the program holds before the call,
`run` is the call, `work` the bytes and operations that one call cannot do
without, `exact` the same result by plain torch in 64 bits.

Kinds:
  step     forward steps of one lattice; "measure" ends the pass as a monitored
           run does, with the conserved functional of the last step and the
           observables
  reverse  exact time reversal of steps made before
  links    forward steps with the gauge links of a vector potential, then the
           conserved functional
  adjoint  the gradient of the transmitted probability with respect to V(z)
  batch    independent (2+1)D lattices of different sizes advanced together,
           then their functionals

Potentials ("coef"): "free" (a mass alone), "vz" (tables of V(z), 3D), "absorb"
(V(z) and absorbing layers; in 2D per-site V and an absorbing frame, complex64),
"site" (a value per site).  "zero": zero values outside the lattice instead of
the periodic wrap.
"""
import math

import numpy as np
import torch

import paper_1309_3452_amd as P

DT2, DT3 = 0.9 / math.sqrt(2.0), 0.9 / math.sqrt(3.0)   # 0.9 x the stability bound
# site positions within a cell of each state array (x, y, z)
OFF3 = ((0., 0., 0.), (.5, .5, 0.), (.5, 0., .5), (0., .5, .5), (0., 0., .5), (.5, .5, .5), (.5, 0., 0.), (0., .5, 0.))
OFF2 = ((0., 0.), (.5, .5), (.5, 0.), (0., .5))
MOST_WORK = 512 ** 3 * 64 * 10      # cells x bytes of a cell's state x steps of the largest listed case


def listed():
    return [
        # a packet on a small plane: every launch is short, so its cost is latency
        dict(name="plane_128_c128", kind="step", ndim=2, dtype="c128", nx=128, ny=128, nz=1, coef="free", zero=False,
             steps=200, measure=False),
        # Klein-step scattering in the plane, a potential per site and an absorbing frame
        dict(name="klein_1024x512_c64", kind="step", ndim=2, dtype="c64", nx=1024, ny=512, nz=1, coef="absorb",
             zero=False, steps=100, measure=False),
        # a large plane of odd width, a potential per site
        dict(name="plane_odd_2047x1531_c64", kind="step", ndim=2, dtype="c64", nx=2047, ny=1531, nz=1, coef="site",
             zero=False, steps=20, measure=False),
        # a small box, many steps
        dict(name="box_64_c64", kind="step", ndim=3, dtype="c64", nx=64, ny=64, nz=64, coef="vz", zero=False,
             steps=100, measure=False),
        # the Klein-step box in 64 bits, monitored
        dict(name="box_256_c128", kind="step", ndim=3, dtype="c128", nx=256, ny=256, nz=256, coef="vz", zero=False,
             steps=10, measure=True),
        # the largest box: the framework's benchmark workload
        dict(name="box_512_c64", kind="step", ndim=3, dtype="c64", nx=512, ny=512, nz=512, coef="vz", zero=False,
             steps=10, measure=False),
        # a ragged box with a potential per site, 64 bits
        dict(name="site_200x168x152_c128", kind="step", ndim=3, dtype="c128", nx=200, ny=168, nz=152, coef="site",
             zero=False, steps=10, measure=False),
        # a box of odd sizes with absorbing layers along z
        dict(name="odd_191x151x127_c64", kind="step", ndim=3, dtype="c64", nx=191, ny=151, nz=127, coef="absorb",
             zero=False, steps=10, measure=False),
        # a box with zero values outside
        dict(name="zero_224x192x256_c64", kind="step", ndim=3, dtype="c64", nx=224, ny=192, nz=256, coef="vz",
             zero=True, steps=10, measure=True),
        # a vector potential
        dict(name="links_256_c64", kind="links", ndim=3, dtype="c64", nx=256, ny=256, nz=256, coef="vz", zero=False,
             steps=5, measure=False),
        # fitting V(z) to a transmitted probability: forward, then the adjoint
        dict(name="adjoint_128_c128", kind="adjoint", ndim=3, dtype="c128", nx=128, ny=128, nz=128, coef="vz",
             zero=False, steps=40, measure=False),
        # many uneven planes at once
        dict(name="batch_15_c64", kind="batch", ndim=2, dtype="c64", count=15, sizes=4, steps=100),
    ]


def _size(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    while True:
        kind = rng.choice(("step", "step", "step", "step", "reverse", "links", "adjoint", "batch"))
        dtype = rng.choice(("c64", "c128"))
        if kind == "batch":
            c = dict(kind=kind, ndim=2, dtype=dtype, count=rng.randint(2, 15), sizes=rng.randint(100, 10 ** 6),
                     steps=_size(rng, 10, 200))
        else:
            ndim = 3 if kind == "adjoint" else rng.choice((2, 3))
            if ndim == 2:
                nx, ny, nz, steps = _size(rng, 32, 4096), _size(rng, 32, 4096), 1, _size(rng, 4, 200)
                coef = rng.choice(("free", "site", "absorb") if dtype == "c64" else ("free", "site"))
            else:
                top = 128 if kind == "adjoint" else 320
                nx, ny, nz = _size(rng, 16, top), _size(rng, 16, top), _size(rng, 16, top)
                steps = _size(rng, 2, 40)
                coef = rng.choice(("vz", "absorb", "site"))
            if kind == "adjoint":
                coef = "vz"
            if kind == "reverse" and coef == "absorb":
                coef = "site"
            zero = kind in ("step", "reverse") and rng.random() < 0.25
            c = dict(kind=kind, ndim=ndim, dtype=dtype, nx=nx, ny=ny, nz=nz, coef=coef, zero=zero, steps=steps,
                     measure=kind == "step" and rng.random() < 0.25)
        w = _cells(c) * _cell_bytes(c) * c["steps"] * (5 if kind == "links" else 10 if kind == "adjoint" else 1)
        if w <= MOST_WORK / 4:
            return c


# ---------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------
def _batch_sizes(c):
    g = np.random.default_rng(c["sizes"])
    return [(int(g.choice(np.arange(64, 1025, 32))), int(g.choice(np.arange(64, 1025, 32)))) for _ in range(c["count"])]


def _cells(c):
    if c["kind"] == "batch":
        return sum(x * y for x, y in _batch_sizes(c))
    return c["nx"] * c["ny"] * c["nz"]


def _cell_bytes(c):
    return (8 if c["ndim"] == 3 else 4) * (8 if c["dtype"] == "c64" else 16)


def _ctype(c):
    return torch.complex64 if c["dtype"] == "c64" else torch.complex128


def _axis(n, off, centre, sigma, k):
    """exp(-d^2 / 4 sigma^2) exp(i k x) along one axis, d the periodic distance to the centre."""
    x = torch.arange(n, dtype=torch.float64, device="cuda") + off
    d = torch.remainder(x - centre + n / 2.0, n) - n / 2.0
    return torch.exp(-d * d / (4.0 * sigma * sigma)) * torch.exp(1j * k * x)


def _packet(g, sizes, m, dtype, dt):
    """A Gaussian packet with the positive-energy spinor of its momentum, its
    place, width and momentum from the generator; sizes (nx, ny[, nz])."""
    nd = len(sizes)
    centre = [float(g.uniform(0.3, 0.7) * n) for n in sizes]
    sigma = [max(2.0, float(g.uniform(0.1, 0.2)) * n) for n in sizes]
    k = [float(g.uniform(-0.2, 0.2)) for _ in sizes]
    k[-1 if nd == 3 else 0] = float(g.uniform(0.3, 0.6))
    E = math.sqrt(m * m + sum(q * q for q in k))
    if nd == 3:
        amps = [1.0, 0.1j, k[2] / (E + m), complex(k[0], k[1]) / (E + m)]
    else:
        amps = [1.0, complex(k[0], k[1]) / (E + m)]
    out = []
    for a, off in enumerate(OFF3 if nd == 3 else OFF2):
        ph = complex(math.cos(E * dt / 2), math.sin(E * dt / 2)) if a < (4 if nd == 3 else 2) else 1.0
        fac = [_axis(n, o, ce, s, q).to(dtype) for n, o, ce, s, q in zip(sizes, off, centre, sigma, k)]
        f = fac[1][:, None] * (fac[0] * (amps[a // 2] * ph))[None, :]
        if nd == 3:
            f = fac[2][:, None, None] * f[None]
        out.append(f)
    s = math.sqrt(sum(float(torch.sum(torch.abs(t).square(), dtype=torch.float64)) for t in out))
    return [t.div_(s) for t in out]


def _v_tables(g, n):
    """A smooth step with some structure, at integer and half-integer z."""
    z = np.arange(n, dtype=np.float64)
    v0, zc = float(g.uniform(0.8, 1.5)), float(g.uniform(0.45, 0.55)) * n
    ripple = 0.05 * g.standard_normal(4)
    f = lambda x: v0 * (1.0 + np.tanh((x - zc) / 4.0)) / 2.0 + sum(
        r * np.cos(2 * math.pi * (q + 1) * x / n) for q, r in enumerate(ripple))
    return f(z), f(z + 0.5)


def _layer(n, off):
    """Absorbing layers at both ends of an axis: W <= 0."""
    x = np.arange(n, dtype=np.float64) + off
    d, width = np.minimum(x, n - x), max(4.0, min(32.0, n / 8.0))
    return np.where(d < width, -0.5 * ((width - d) / width) ** 2, 0.0)


def _v_site(g, sizes, real):
    """Smooth bumps plus a little noise, at every array's own sites."""
    nd = len(sizes)
    bumps = [(float(g.uniform(-1, 1)), [float(g.uniform(0, n)) for n in sizes],
              [max(2.0, float(g.uniform(1 / 16, 1 / 4)) * n) for n in sizes]) for _ in range(4)]
    tg = torch.Generator(device="cuda").manual_seed(int(g.integers(1 << 40)))
    out = []
    for off in (OFF3 if nd == 3 else OFF2):
        v = 0.02 * torch.randn(tuple(reversed(sizes)), generator=tg, device="cuda", dtype=real)
        for amp, ce, s in bumps:
            fac = [torch.abs(_axis(n, o, c0, w / math.sqrt(2.0), 0.0)).to(real)
                   for n, o, c0, w in zip(sizes, off, ce, s)]
            f = amp * fac[1][:, None] * fac[0][None, :]
            v += fac[2][:, None, None] * f[None] if nd == 3 else f
        out.append(v)
    return out


def _links(g, c):
    """Gauge links of a smooth periodic vector potential: exp(-i a_j d_j) per
    half-link, 24 (3D) or 8 (2D) arrays."""
    sizes, nd = (c["nx"], c["ny"], c["nz"])[:c["ndim"]], c["ndim"]
    ph, amp = g.uniform(0, 2 * math.pi, 6), 0.05
    dirs = ((2, .5), (2, -.5), (0, .5), (0, -.5), (1, .5), (1, -.5)) if nd == 3 else ((0, .5), (0, -.5), (1, .5), (1, -.5))
    out = []
    for off in (OFF3[:4] if nd == 3 else OFF2[:2]):
        for ax, d in dirs:
            x = [torch.arange(n, dtype=torch.float64, device="cuda") + o + (0.5 * d if q == ax else 0.0)
                 for q, (n, o) in enumerate(zip(sizes, off))]
            u, w = (1, 2 if nd == 3 else 0) if ax == 0 else (0, 2 if nd == 3 else 1) if ax == 1 else (0, 1)
            su = torch.sin(2 * math.pi * x[u] / sizes[u] + ph[2 * ax])
            sw = torch.cos(2 * math.pi * x[w] / sizes[w] + ph[2 * ax + 1])
            shape = lambda q: [-1 if (nd - 1 - t) == q else 1 for t in range(nd)]
            a = amp * d * su.view(shape(u)) * sw.view(shape(w))
            out.append(torch.polar(torch.ones((), dtype=torch.float64, device="cuda"), -a).to(_ctype(c))
                       .expand(tuple(reversed(sizes))).contiguous())
    return out


def _inputs(c, seed):
    """Everything that a case's program is given, from the seed alone."""
    g = np.random.default_rng([13093452, int(seed)])
    real = torch.float32 if c["dtype"] == "c64" else torch.float64
    if c["kind"] == "batch":
        lats = []
        for nx, ny in _batch_sizes(c):
            m = float(g.uniform(0.0, 1.0))
            lats.append(dict(nx=nx, ny=ny, m=m, v_site=_v_site(g, (nx, ny), real),
                             state=_packet(g, (nx, ny), m, _ctype(c), DT2)))
        return dict(lats=lats)
    sizes = (c["nx"], c["ny"], c["nz"])[:c["ndim"]]
    q = dict(m=0.0 if c["coef"] == "free" else 0.5, v_int=None, w_int=None, v_site=None, w_site=None, links=None)
    q["state"] = _packet(g, sizes, q["m"], _ctype(c), DT3 if c["ndim"] == 3 else DT2)
    if c["ndim"] == 3 and c["coef"] in ("vz", "absorb"):
        q["v_int"], q["v_half"] = _v_tables(g, c["nz"])
        if c["coef"] == "absorb":
            q["w_int"], q["w_half"] = _layer(c["nz"], 0.0), _layer(c["nz"], 0.5)
    elif c["coef"] in ("site", "absorb"):
        q["v_site"] = _v_site(g, sizes, real)
        if c["coef"] == "absorb":
            q["w_site"] = [torch.as_tensor(_layer(c["nx"], o[0]), device="cuda").expand(c["ny"], c["nx"]).contiguous()
                           for o in OFF2]
    if c["kind"] == "links":
        q["links"] = _links(g, c)
    return q


# ---------------------------------------------------------------------------
# the framework
# ---------------------------------------------------------------------------
def prepare(case, seed):
    q = _inputs(case, seed)
    if case["kind"] == "batch":
        return dict(case=case, batch=P.BatchedLattices(q["lats"], dtype=_ctype(case), dt=DT2))
    sizes = (case["nx"], case["ny"], case["nz"])[:case["ndim"]]
    lat = P.Lattice(sizes, dtype=_ctype(case), dt=DT3 if case["ndim"] == 3 else DT2, zero_bc=case["zero"])
    s = dict(case=case, lat=lat)
    if case["kind"] == "adjoint":
        s.update(state0=q["state"], m=q["m"], v_int=q["v_int"], v_half=q["v_half"])
        return s
    if q["v_site"] is not None:
        lat.set_fields(q["m"], q["v_site"], q["w_site"])
    else:
        lat.set_potential_z(q["m"], q["v_int"], q.get("v_half"))
        if q["w_int"] is not None:
            lat.set_absorber_z(q["w_int"], q["w_half"])
    if q["links"] is not None:
        lat.set_links(q["links"])
    lat.load(q["state"])
    return s


def run(state):
    c = state["case"]
    if c["kind"] == "batch":
        b = state["batch"]
        b.run(c["steps"])
        return [b.state(k) for k in range(b.count)], np.array(b.norms())
    lat = state["lat"]
    if c["kind"] == "adjoint":
        loss, dvi, dvh = P.potential_gradient(lat, state["state0"], state["m"], state["v_int"], state["v_half"],
                                              c["steps"], c["nz"] / 2.0)
        return loss, dvi, dvh, list(lat.state())
    if c["kind"] == "reverse":
        lat.reverse(c["steps"])
        return list(lat.state())
    if c["kind"] == "links":
        lat.step(c["steps"])
        return list(lat.state()), lat.norm()
    if c["measure"]:
        e = lat.step_norm(c["steps"])
        return list(lat.state()), e, lat.observables(_z0(c))
    lat.step(c["steps"])
    return list(lat.state())


def _z0(c):
    return (c["nz"] if c["ndim"] == 3 else c["nx"]) / 2.0


def work(case):
    """Bytes: the state read once and written once, and each coefficient or link
    read once, per call; operations: 4 (2D) or 8 (3D) updates per cell and step,
    each a difference term of 10 (6) real operations per component and an update
    of 16 in all, links adding a complex product per neighbour."""
    c, cells, b = case, _cells(case), 8 if case["dtype"] == "c64" else 16
    narr, near = (8, 6) if c["ndim"] == 3 else (4, 4)
    site = c["kind"] == "batch" or c["coef"] == "site" or (c["coef"] == "absorb" and c["ndim"] == 2)
    bytes_ = cells * narr * (2 * b + (8 if site else 0))
    flops = cells * c["steps"] * narr * (16 + 2 * near + 4)
    if c["kind"] == "links":
        bytes_ += cells * (24 if c["ndim"] == 3 else 8) * b
        flops += cells * c["steps"] * narr * near * 6
    if c["kind"] == "adjoint":      # forward, then state and adjoint backward and the gradient's products
        flops *= 4
    return dict(bytes=bytes_, flops=flops)


# ---------------------------------------------------------------------------
# the same by plain torch, 64 bits
# ---------------------------------------------------------------------------
# S_X of the A,B (u) arrays: for each neighbour direction the array reached, its
# cell offset (x, y, z) and its factor (axis of r, complex coefficient).  The
# C,D (v) arrays' terms are the negative adjoint of these.
TERMS3 = (
    ((0, (0, 0, 0), 2, 1), (0, (0, 0, -1), 2, -1), (2, (0, 0, 0), 0, 1), (2, (-1, 0, 0), 0, -1),
     (3, (0, 0, 0), 1, -1j), (3, (0, -1, 0), 1, 1j)),
    ((1, (0, 0, 0), 2, 1), (1, (0, 0, -1), 2, -1), (3, (1, 0, 0), 0, 1), (3, (0, 0, 0), 0, -1),
     (2, (0, 1, 0), 1, -1j), (2, (0, 0, 0), 1, 1j)),
    ((2, (0, 0, 1), 2, -1), (2, (0, 0, 0), 2, 1), (0, (1, 0, 0), 0, 1), (0, (0, 0, 0), 0, -1),
     (1, (0, 0, 0), 1, 1j), (1, (0, -1, 0), 1, -1j)),
    ((3, (0, 0, 1), 2, -1), (3, (0, 0, 0), 2, 1), (1, (0, 0, 0), 0, 1), (1, (-1, 0, 0), 0, -1),
     (0, (0, 1, 0), 1, 1j), (0, (0, 0, 0), 1, -1j)))
TERMS2 = (
    ((0, (0, 0), 0, 1), (0, (-1, 0), 0, -1), (1, (0, 0), 1, -1j), (1, (0, -1), 1, 1j)),
    ((1, (1, 0), 0, 1), (1, (0, 0), 0, -1), (0, (0, 1), 1, -1j), (0, (0, 0), 1, 1j)))


class _Exact:
    """The scheme on one lattice; f: its arrays in complex128."""

    def __init__(self, f, r, theta, zero=False, links=None):
        self.f, self.r, self.zero, self.links = list(f), r, zero, links
        self.terms = TERMS3 if len(f) == 8 else TERMS2
        self.h = len(f) // 2
        self.theta = theta          # one per array, broadcastable
        self.alpha = [(1 - 1j * t) / (1 + 1j * t) for t in theta]
        self.beta = [1 / (1 + 1j * t) for t in theta]

    def at(self, x, off):
        """x at the cell displaced by off."""
        nd = x.dim()
        for ax, o in enumerate(off):
            if o:
                d = nd - 1 - ax
                x = torch.roll(x, -o, d)
                if self.zero:
                    x.select(d, x.shape[d] - 1 if o > 0 else 0).zero_()
        return x

    def s_first(self, a):
        out = 0
        for t, (b, off, ax, k) in enumerate(self.terms[a]):
            v = self.at(self.f[self.h + b], off)
            if self.links is not None:
                v = self.links[len(self.terms[a]) * a + t].to(torch.complex128) * v
            out = out + (k * self.r[ax]) * v
        return out

    def s_second(self, b):
        out = 0
        for a, row in enumerate(self.terms):
            for t, (bb, off, ax, k) in enumerate(row):
                if bb == b:
                    v = self.f[a]
                    if self.links is not None:
                        v = self.links[len(row) * a + t].to(torch.complex128).conj() * v
                    out = out - (complex(k).conjugate() * self.r[ax]) * self.at(v, tuple(-o for o in off))
        return out

    def half(self, second, back=False):
        new = []
        for q in range(self.h):
            s = self.s_second(q) if second else self.s_first(q)
            a = self.h + q if second else q
            new.append((self.f[a] + self.beta[a] * s) / self.alpha[a] if back
                       else self.alpha[a] * self.f[a] - self.beta[a] * s)
        self.f[self.h if second else 0:2 * self.h if second else self.h] = new

    def step(self, n):
        for _ in range(n):
            self.half(False)
            self.half(True)

    def reverse(self, n):
        for _ in range(n):
            self.half(True, back=True)
            self.half(False, back=True)

    def norms(self):
        """The functional in both forms and the plain norm."""
        p = sum(torch.sum(torch.abs(x).square()) for x in self.f)
        e0 = p - sum(torch.sum((self.f[a].conj() * self.s_first(a)).real) for a in range(self.h))
        e1 = p + sum(torch.sum((self.f[self.h + b].conj() * self.s_second(b)).real) for b in range(self.h))
        return [float(e0), float(e1), float(p)]

    def observables(self, z0):
        nd = self.f[0].dim()
        out = np.zeros(9)
        for a, x in enumerate(self.f):
            p, off = torch.abs(x).square(), (OFF3 if nd == 3 else OFF2)[a]
            sums = []
            for ax in range(nd):
                s = p.sum(dim=[d for d in range(nd) if d != nd - 1 - ax])
                pos = torch.arange(s.numel(), dtype=torch.float64, device="cuda") + off[ax]
                sums.append((float((pos * s).sum()), float(s[pos >= z0].sum())))
            out[0] += sums[2 if nd == 3 else 0][1]
            for ax in range(nd):
                out[1 + ax] += sums[ax][0]
            out[1 + nd] += float(p.sum())
            out[2 + nd + a // 2] += float(p.sum())
        return tuple(float(v) for v in out)


def _theta(c, q, dt):
    """Theta of every array, 64 bits: per site, or per plane of z."""
    narr = 8 if c["ndim"] == 3 else 4
    out = []
    for a in range(narr):
        sm = q["m"] if a < narr // 2 else -q["m"]
        if q["v_site"] is not None:
            t = sm + q["v_site"][a].double()
            if q["w_site"] is not None:
                t = t + 1j * q["w_site"][a].double()
        elif q["v_int"] is not None:
            half = a // 2 in (1, 2)
            v = q["v_half"] if half else q["v_int"]
            t = sm + torch.as_tensor(v, device="cuda")
            if q["w_int"] is not None:
                t = t + 1j * torch.as_tensor(q["w_half"] if half else q["w_int"], device="cuda")
            t = t.view(-1, 1, 1)
        else:
            t = torch.full((), sm, dtype=torch.float64, device="cuda")
        out.append(0.5 * dt * t)
    return out


def exact(case, seed):
    c, q = case, _inputs(case, seed)
    if c["kind"] == "batch":
        states, norms = [], []
        for L in q["lats"]:
            th = [0.5 * DT2 * ((L["m"] if a < 2 else -L["m"]) + L["v_site"][a].double()) for a in range(4)]
            x = _Exact([t.to(torch.complex128) for t in L["state"]], (DT2, DT2), th)
            x.step(c["steps"])
            states.append(x.f)
            norms.append(x.norms())
        return states, np.array(norms)
    dt = DT3 if c["ndim"] == 3 else DT2
    f = [t.to(torch.complex128) for t in q.pop("state")]
    if c["kind"] == "adjoint":
        vi, vh = (torch.tensor(q[k], device="cuda", requires_grad=True) for k in ("v_int", "v_half"))
        theta = [0.5 * dt * ((q["m"] if a < 4 else -q["m"]) + (vh if a // 2 in (1, 2) else vi)).view(-1, 1, 1)
                 for a in range(8)]
        x = _Exact(f, (dt,) * 3, theta)
        x.step(c["steps"])
        z = torch.arange(c["nz"], dtype=torch.float64, device="cuda")
        loss = sum(torch.sum(torch.view_as_real(t[(z + OFF3[a][2]) >= c["nz"] / 2.0]).square())
                   for a, t in enumerate(x.f))
        gi, gh = torch.autograd.grad(loss, (vi, vh))
        return float(loss), gi, gh, f
    x = _Exact(f, (dt,) * c["ndim"], _theta(c, q, dt), c["zero"], q["links"])
    del f
    if c["kind"] == "reverse":
        x.reverse(c["steps"])
        return x.f
    x.step(c["steps"])
    if c["kind"] == "links":
        return x.f, tuple(x.norms())
    if c["measure"]:
        e = x.norms()
        return x.f, torch.tensor([e[1], e[2]], dtype=torch.float64), x.observables(_z0(c))
    return x.f
