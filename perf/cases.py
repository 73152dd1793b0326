"""Workloads that a user of the particle-mesh framework runs, through its public Python entry points.

A case is a dict of plain values; `listed()` gives the fixed ones, `draw(rng)` one more of the same
ranges.  `prepare` makes what the program holds before the call (particles on the GPU, a context),
`run` is one pass, `work` the bytes and operations it cannot do without, `exact` the same outputs from a
plain torch implementation of the equations in 64 bits.

Kinds of pass:
  load    particles from device arrays into a context, a few steps, particles and fields back: a short
          run as a parameter scan or a test makes it (small meshes: launches and latency count);
  evolve  a running simulation advances to its next output: some steps on a loaded context, then the
          particles and the metric fields are copied out (with the learned closure on where asked);
  force   the closure's training labels: particles of another density than the mesh are loaded, the
          metric is solved once and grad phi is gathered at the particles;
  train   one iteration of the closure's training: augmentation, load, deposit, solve, network forward,
          loss, backward, Adam;
  power   the matter power spectrum of the loaded particles;
  fft     3D transforms of a few fields there and back through the entry point that allocates nothing.
"""
import math

import numpy as np
import torch

from paper_2607_17929_amd import pm as gpm

FIELDS = {"newtonian": ("phi",), "scalar": ("phi", "chi"), "full": ("phi", "chi", "bx", "by", "bz")}
MPCH_PER_CELL = 4.0  # the clustered workloads' mesh spacing
SYM = ((0, 0), (0, 1), (0, 2), (1, 1), (1, 2), (2, 2))
NPARAM = 9971        # weights and biases of the closure's three layers
LAYERS = ((4, 16), (16, 16), (16, 3))


def listed():
    return [
        # the smallest call: a Newtonian scan point on the smallest mesh, an odd particle count
        dict(name="newton_16", kind="load", n=16, np=1001, physics="newtonian", precision="fp64", steps=4, a=0.1,
             dtau=0.01),
        # the repository's 32^3 Zel'dovich workload: ten FP64 scalar steps, a = 0.02 -> 0.05
        dict(name="zeldovich_32", kind="load", n=32, np=32768, physics="scalar", precision="fp64", steps=10, a=0.02,
             dtau=0.0581),
        # a small box with a hot second species, reproducible bit for bit, the paper's 12-FFT route; ragged counts
        dict(name="species_64", kind="load", n=64, np=250007, physics="full", precision="fp32", steps=5, a=0.1,
             dtau=0.01, parabolic=True, deterministic=True, np2=50021),
        # the 256^3 k T(k)-sized workload, full physics, FP32, between two outputs
        dict(name="evolve_256", kind="evolve", n=256, np=256 ** 3, physics="full", precision="fp32", steps=4, a=0.1,
             dtau=0.01),
        # the FP64 path with the parabolic route, ragged count
        dict(name="evolve_256_fp64", kind="evolve", n=256, np=15999989, physics="full", precision="fp64", steps=2,
             a=0.1, dtau=0.01, parabolic=True),
        # the closure's application: corrected scalar steps of a clustered box
        dict(name="closure_256", kind="evolve", n=256, np=256 ** 3, physics="scalar", precision="fp32", steps=3, a=0.5,
             dtau=0.01, clustered=True, closure=True),
        # the benchmark's size: 512^3 clustered, full physics, FP32
        dict(name="evolve_512", kind="evolve", n=512, np=512 ** 3, physics="full", precision="fp32", steps=4, a=0.5,
             dtau=0.01, clustered=True),
        # labels of the closure's training: 128^3 particles on the 2x mesh
        dict(name="force_256", kind="force", n=256, np=128 ** 3, physics="scalar", precision="fp32", a=0.3,
             clustered=True),
        # one training iteration on the 1x mesh of the training boxes
        dict(name="train_128", kind="train", n=128, np=128 ** 3, physics="scalar", precision="fp32", a=0.3,
             clustered=True),
        # P(k) of a finished run on the measurement mesh
        dict(name="power_512", kind="power", n=512, np=512 ** 3, physics="newtonian", precision="fp32", a=0.5,
             clustered=True),
        # transforms in a loop that may not allocate
        dict(name="fft_128", kind="fft", n=128, precision="fp32", fields=2),
    ]


def draw(rng):
    kind = rng.choice(["load", "load", "evolve", "evolve", "force", "train", "power", "fft"])
    if kind == "fft":
        return dict(kind=kind, n=2 ** rng.randint(4, 7), precision=rng.choice(["fp32", "fp64"]), fields=rng.randint(1, 12))
    top = {"load": 7, "evolve": 9, "force": 8, "train": 7, "power": 9}[kind]
    low = {"load": 4, "evolve": 7, "force": 5, "train": 5, "power": 5}[kind]
    n = 2 ** rng.randint(low, top)
    # particles per cell from one in eight to one and a half, odd counts among them
    count = int(n ** 3 * math.exp(rng.uniform(math.log(0.125), math.log(1.5 if n < 512 else 1.0))))
    c = dict(kind=kind, n=n, np=max(count | 1, 1), a=round(math.exp(rng.uniform(math.log(0.05), math.log(0.5))), 4),
             clustered=rng.random() < 0.5)
    if kind in ("load", "evolve"):
        c["physics"] = rng.choice(["newtonian", "scalar", "full", "full"])
        # Newtonian runs are the plain comparison and take 64 bits; the largest mesh has room for 32
        if n > 256 and c["physics"] == "newtonian":
            c["physics"] = "scalar"
        c["precision"] = "fp64" if c["physics"] == "newtonian" or (n <= 256 and rng.random() < 0.3) else "fp32"
        c["steps"] = rng.randint(2, 8) if kind == "load" else rng.randint(2, 4)
        c["dtau"] = 0.01 if n > 128 else 0.004
        if c["physics"] == "full":
            c["parabolic"] = rng.random() < 0.5
        if rng.random() < 0.25:
            c["deterministic"] = True
        if kind == "load" and rng.random() < 0.3:
            c["np2"] = max(count // 5, 1) | 1
        if kind == "evolve" and n <= 256 and c["precision"] == "fp32" and rng.random() < 0.25:
            c["closure"] = True
    else:
        c["physics"] = "newtonian" if kind == "power" else "scalar"
        c["precision"] = "fp32"
    return c


# ---------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------

def _box(case):
    return MPCH_PER_CELL * case["n"]


def _h0(box):
    return box / 2997.92458


def _tau(case):
    return 2.0 * math.sqrt(case["a"]) / _h0(_box(case))


def particles(case, seed):
    """(pos [np][3] float64, u [np][3] in the case's precision) on the GPU, ordered by lattice site as a
    generator of initial conditions leaves them: a displaced lattice with P(k) ~ k^-2 (rms 0.2 spacings at
    a = 0.02, growing with a), velocities of the growing mode; where `clustered`, the displacement is
    capped and a quarter of the lattice is drawn together into clumps with random motions, so that cells
    hold from none to hundreds of particles."""
    g = torch.Generator(device="cuda").manual_seed(1000 + seed)
    count = case["np"]
    m = max(2, round(count ** (1.0 / 3.0)))
    while m ** 3 < count:
        m += 1
    clustered = bool(case.get("clustered"))
    dk = torch.fft.rfftn(torch.randn((m, m, m), generator=g, device="cuda"))
    kz = torch.fft.fftfreq(m, 1.0 / m, device="cuda")[:, None, None]
    ky = torch.fft.fftfreq(m, 1.0 / m, device="cuda")[None, :, None]
    kx = torch.arange(m // 2 + 1, device="cuda", dtype=torch.float32)[None, None, :]
    k2 = kx * kx + ky * ky + kz * kz
    k2[0, 0, 0] = 1.0
    amp = torch.where(k2 < (0.5 * m) ** 2, k2 ** -1.5, torch.zeros_like(k2))
    amp[0, 0, 0] = 0.0
    dk *= amp  # sqrt(P) / k^2
    del amp, k2
    psi = [torch.fft.irfftn(1j * k * dk, s=(m, m, m)).reshape(-1) for k in (kx, ky, kz)]
    del dk
    # lattice spacings: the linear displacement, and how much of it the positions take
    rms = math.sqrt(sum(float((p * p).mean(dtype=torch.float64)) for p in psi)) or 1.0
    lin = 0.2 * case["a"] / 0.02
    site = torch.arange(count, device="cuda", dtype=torch.int64)
    if count < m ** 3:
        site = (site * (m ** 3)) // count
    psi = [(p * (lin / rms))[site] for p in psi]
    take = min(1.0, 2.0 / lin) if clustered else 1.0
    pos = torch.empty((count, 3), dtype=torch.float64, device="cuda")
    u = torch.empty((count, 3), dtype=torch.float64, device="cuda")
    hc = 2.0 / _tau(case)
    q = [site % m, (site // m) % m, site // (m * m)]
    del site
    pull = None
    if clustered:
        # blocks of 16^3 and 8^3 sites collapse towards their centres
        pull = torch.zeros(count, dtype=torch.int64, device="cuda")
        for b, share in ((8, 0.22), (16, 0.08)):
            nb = (m + b - 1) // b
            falls = torch.rand(nb ** 3, generator=g, device="cuda") < share
            hit = falls[((q[2] // b) * nb + q[1] // b) * nb + q[0] // b]
            pull = torch.where(hit, torch.full_like(pull, b), pull)
            del hit
        size = pull.clamp(min=1)
        off = [(qi % size).double() - 0.5 * (size - 1).double() for qi in q]
        r = torch.sqrt(off[0] ** 2 + off[1] ** 2 + off[2] ** 2)
        # radius r' = 0.7 r^2 / (b / 2)^1.5: a cusp at the centre
        shrink = torch.where(pull > 0, 0.7 * r / (0.5 * size.double()) ** 1.5, torch.ones_like(r)).clamp(max=1.0)
        del r, size
    for d in range(3):
        x = q[d].double() + 0.5 + take * psi[d].double()
        v = hc * psi[d].double() / m
        if pull is not None:
            x = x - off[d] * (1.0 - shrink) + torch.where(
                pull > 0, 0.3 * torch.randn(count, generator=g, device="cuda", dtype=torch.float64), torch.zeros_like(x))
            v = v + torch.where(pull > 0, (hc * 5.0 / m) * torch.randn(count, generator=g, device="cuda",
                                                                         dtype=torch.float64), torch.zeros_like(x))
        x = x / m
        x = x - torch.floor(x)
        pos[:, d] = torch.where(x >= 1.0, torch.zeros_like(x), x)
        u[:, d] = case["a"] * v
    return pos, (u if case["precision"] == "fp64" else u.float())


def second_species(case, seed):
    """Hot particles: uniform positions, |u| = 2 a in random directions."""
    g = torch.Generator(device="cuda").manual_seed(5000 + seed)
    pos = torch.rand((case["np2"], 3), generator=g, device="cuda", dtype=torch.float64)
    u = torch.randn((case["np2"], 3), generator=g, device="cuda", dtype=torch.float64)
    u = u * (2.0 * case["a"] / u.norm(dim=1, keepdim=True))
    return pos, (u if case["precision"] == "fp64" else u.float())


def weights(seed, last=0.1):
    """The closure's parameter vector (He-style, small last layer)."""
    r = np.random.default_rng(77 + seed)
    out = []
    for li, (ci, co) in enumerate(LAYERS):
        out.append(r.standard_normal(co * ci * 27) * math.sqrt(2.0 / (ci * 27)) * (last if li == 2 else 1.0))
        out.append(0.01 * r.standard_normal(co))
    return torch.tensor(np.concatenate(out), dtype=torch.float32, device="cuda")


def training_rest(case, seed):
    """Target forces, Adam's moments of a run under way, the symmetry of this iteration."""
    g = torch.Generator(device="cuda").manual_seed(9000 + seed)
    target = 0.1 * torch.randn((case["np"], 3), generator=g, device="cuda")
    m = 1e-4 * torch.randn(NPARAM, generator=g, device="cuda")
    v = 1e-6 * (1.0 + torch.rand(NPARAM, generator=g, device="cuda"))
    r = np.random.default_rng(seed)
    return target, m, v, [int(p) for p in r.permutation(3)], int(r.integers(8))


def _context(case):
    return gpm.PMContext(case["n"], case["np"], _box(case), physics=case["physics"], precision=case["precision"],
                         closure=case["kind"] == "train" or bool(case.get("closure")),
                         b_route="parabolic" if case.get("parabolic") else "elliptic",
                         n_particles_2=case.get("np2", 0), mass_fraction_2=0.1 if case.get("np2") else 0.0,
                         deterministic=bool(case.get("deterministic")))


def prepare(case, seed):
    s = {"case": case}
    if case["kind"] == "fft":
        g = torch.Generator(device="cuda").manual_seed(seed)
        s["x"] = [torch.randn((case["n"],) * 3, generator=g, device="cuda",
                              dtype=torch.float64 if case["precision"] == "fp64" else torch.float32)
                  for _ in range(case["fields"])]
        return s
    pos, u = particles(case, seed)
    ctx = s["ctx"] = _context(case)
    s["tau"] = _tau(case)
    if case["kind"] in ("evolve", "power"):
        ctx.init_particles(pos, u, s["tau"])
        if case.get("closure"):
            ctx.closure_set_params(weights(seed))
            ctx.closure_enable(True)
        if case["kind"] == "evolve":
            s["dtau"] = case["dtau"] * s["tau"]
            ctx.step(s["dtau"])  # the start-up solve
        ctx.sync()
        return s
    s["pos"], s["u"] = pos, u
    if case["kind"] == "load":
        s["dtau"] = case["dtau"] * s["tau"]
        if case.get("np2"):
            s["pos2"], s["u2"] = second_species(case, seed)
    elif case["kind"] == "train":
        s["target"], s["m"], s["v"], s["perm"], s["flip"] = training_rest(case, seed)
        s["params"], s["it"] = weights(seed), 1000
        s["aug"] = (torch.empty_like(pos), torch.empty_like(u), torch.empty_like(s["target"]))
        s["dpred"] = torch.empty_like(s["target"])
        ctx.closure_set_params(s["params"])
    return s


# ---------------------------------------------------------------------------
# one pass
# ---------------------------------------------------------------------------

def _outputs(ctx, case):
    pos, u = ctx.get_particles(device=True)
    out = {"pos": pos, "u": u}
    for f in FIELDS[case["physics"]]:
        out[f] = ctx.get_field(f, device=True)
    return out


def run(s):
    case, kind = s["case"], s["case"]["kind"]
    if kind == "fft":
        k = [gpm.fft_noalloc(x, case["n"], 1, case["precision"]) for x in s["x"]]
        return {"k": k, "x": [gpm.fft_noalloc(f, case["n"], -1, case["precision"]) for f in k]}
    ctx = s["ctx"]
    if kind == "evolve":
        for _ in range(case["steps"]):
            ctx.step(s["dtau"])
        return _outputs(ctx, case)
    if kind == "load":
        ctx.init_particles(s["pos"], s["u"], s["tau"])
        if case.get("np2"):
            ctx.init_particles_2(s["pos2"], s["u2"])
        for _ in range(case["steps"]):
            ctx.step(s["dtau"])
        return _outputs(ctx, case)
    if kind == "force":
        ctx.init_particles(s["pos"], s["u"], s["tau"])
        ctx.deposit()
        ctx.solve_metric(0.0)
        return {"g": ctx.gather_grad_phi()}
    if kind == "power":
        # FP32 accuracy, as the mesh it comes from
        k, p, modes = ctx.power_spectrum()
        return {"k": k, "p": p.astype(np.float32), "modes": modes.astype(np.int64)}
    pos, u, target = ctx.cube_symmetry(s["pos"], s["u"], s["target"], s["perm"], s["flip"], out=s["aug"])
    ctx.init_particles(pos, u, s["tau"])
    ctx.deposit()
    ctx.solve_metric(0.0)
    ctx.closure_forward(False)
    loss, power, _ = ctx.closure_loss(target, s["dpred"])
    grad = ctx.closure_backward(s["dpred"])
    ctx.closure_adam(s["params"], s["m"], s["v"], grad, s["it"], 1e-3)
    s["it"] += 1
    return {"loss": loss, "power": power, "dpred": s["dpred"], "grad": grad, "params": s["params"], "m": s["m"],
            "v": s["v"]}


# ---------------------------------------------------------------------------
# what a pass cannot do without
# ---------------------------------------------------------------------------

def work(case):
    """Bytes: per step every particle's position and momentum and every field and mode of the metric's
    state once in and once out; then the outputs.  Operations: the transforms (5/2 N log2 N each, real to
    complex), 40 per particle and mesh quantity deposited or gathered, and the network's products."""
    n = case["n"]
    n3, rs = n ** 3, 8 if case["precision"] == "fp64" else 4
    half = n * n * (n // 2 + 1) * 2 * rs
    fft = 2.5 * n3 * math.log2(n3)
    if case["kind"] == "fft":
        return {"bytes": 2 * (n3 * rs + half) * case["fields"], "flops": 2 * fft * case["fields"]}
    npart = case["np"] + case.get("np2", 0)
    part = npart * (24 + 3 * rs)
    nf = len(FIELDS[case["physics"]])
    ffts = {"newtonian": 2, "scalar": 9, "full": 12 if case.get("parabolic") else 15}[case["physics"]]
    conv = 2.0 * 27 * n3 * sum(ci * co for ci, co in LAYERS)
    if case["kind"] == "power":
        return {"bytes": npart * 24 + 24 * (n // 2), "flops": fft + 40.0 * npart}
    if case["kind"] == "force":
        return {"bytes": part + npart * 3 * rs, "flops": 2 * ffts * fft + 40.0 * npart * 14}
    if case["kind"] == "train":
        return {"bytes": 2 * part + 4 * npart * 12 + 6 * 4 * NPARAM,
                "flops": 2 * ffts * fft + 40.0 * npart * 20 + 3 * conv}
    quantities = {"newtonian": 2, "scalar": 18, "full": 30}[case["physics"]]
    flops = case["steps"] * (ffts * fft + 40.0 * npart * quantities + (conv if case.get("closure") else 0.0))
    metric = {"newtonian": 2, "scalar": 6, "full": 9}[case["physics"]] * n3 * rs
    if case["physics"] == "full":
        metric += 8 * half
    steps = case["steps"] * (2 * part + metric)
    return {"bytes": steps + 2 * part + (part if case["kind"] == "load" else 0) + nf * n3 * rs, "flops": flops}


# ---------------------------------------------------------------------------
# the same in 64 bits: the equations written out in torch
# ---------------------------------------------------------------------------

CHUNK = 1 << 24


def _ftn(f):
    return torch.fft.rfftn(f)


def _shift(f, axis, d):
    return torch.roll(f, -d, dims=axis)


class Plain:
    """The particle-mesh step in float64 on [z][y][x] arrays, plain torch."""

    def __init__(self, case, sets, masses):
        self.n, self.physics, self.case = case["n"], case["physics"], case
        self.h0, self.tau = _h0(_box(case)), _tau(case)
        self.sets = [(p.double(), u.double()) for p, u in sets]
        self.w = masses
        self.phi = self.chi = None
        self.delta, self.dtau_last, self.last = None, 0.0, 0.0
        self.h = self.a2b = None
        m = torch.fft.fftfreq(self.n, 1.0 / self.n, device="cuda", dtype=torch.float64)
        kt = 2.0 * self.n * torch.sin(math.pi * m / self.n)
        half = torch.arange(self.n // 2 + 1, device="cuda", dtype=torch.float64)
        self.kt = (2.0 * self.n * torch.sin(math.pi * half / self.n)[None, None, :], kt[None, :, None],
                   kt[:, None, None])
        self.k2 = self.kt[0] ** 2 + self.kt[1] ** 2 + self.kt[2] ** 2
        keep = torch.ones(self.n, dtype=torch.bool, device="cuda")
        keep[self.n // 2] = False
        self.mask = keep[:, None, None] & keep[None, :, None] & (half < self.n // 2)[None, None, :]
        self.mask[0, 0, 0] = False
        self.safe = self.k2.clone()
        self.safe[0, 0, 0] = 1.0

    def a_of(self, tau):
        return (0.5 * self.h0 * tau) ** 2

    def corners(self, p):
        s = p * self.n
        fl = torch.floor(s)
        f = s - fl
        i = fl.long() & (self.n - 1)
        for c in range(8):
            idx = 0
            w = 1.0
            for d, bit in ((2, c >> 2), (1, (c >> 1) & 1), (0, c & 1)):
                idx = idx * self.n + ((i[:, d] + bit) & (self.n - 1))
                w = w * (f[:, d] if bit else 1.0 - f[:, d])
            yield idx, w

    def spread(self, pos, values):
        """CIC sums of the functions in `values` (chunk slice -> [columns]) over the particles."""
        out = None
        for b in range(0, pos.shape[0], CHUNK):
            sl = slice(b, min(b + CHUNK, pos.shape[0]))
            q = values(sl)
            if out is None:
                out = torch.zeros((len(q), self.n ** 3), dtype=torch.float64, device="cuda")
            for idx, w in self.corners(pos[sl]):
                for c, v in enumerate(q):
                    out[c].index_add_(0, idx, w * v)
        return out.reshape(-1, self.n, self.n, self.n)

    def gather(self, fields, p):
        out = [0.0] * len(fields)
        for idx, w in self.corners(p):
            for c, f in enumerate(fields):
                out[c] = out[c] + w * f.reshape(-1)[idx]
        return out

    def grad(self, f):
        return [(_shift(f, ax, 1) - _shift(f, ax, -1)) * (0.5 * self.n) for ax in (2, 1, 0)]

    def deposit(self):
        a = self.a_of(self.tau)
        self.dep = 0.0
        for (pos, u), w in zip(self.sets, self.w):
            def values(sl, u=u, w=w):
                if self.physics == "newtonian":
                    return [torch.full_like(u[sl, 0], a * w)]
                v = u[sl]
                e = torch.sqrt(a * a + (v * v).sum(1))
                return [w * e] + [w * v[:, d] for d in range(3)] + [w * v[:, i] * v[:, j] / e for i, j in SYM]
            self.dep = self.dep + self.spread(pos, values)

    def one_solve(self, phi1, chi1, phidot, inv_dt, incr, elliptic):
        n = self.n
        a, hc = self.a_of(self.tau), 2.0 / self.tau
        eb = 1.5 * self.h0 ** 2 / a
        f2 = 0.1 if len(self.sets) > 1 else 0.0
        kap = 1.5 * self.h0 ** 2 * n ** 3 * (1.0 - f2) / self.sets[0][0].shape[0] / (a * a)
        E = kap * self.dep[0]
        if self.physics == "newtonian":
            return torch.fft.irfftn(_ftn(E - eb) / -self.safe * (self.k2 > 0), s=(n,) * 3), None, None, None
        zero = torch.zeros_like(E)
        p, c = (phi1, chi1) if phi1 is not None else (zero, zero)
        pd = phidot if phidot is not None else 0.0
        gp, gc = self.grad(p), self.grad(c)
        w = 2.0 * p - c
        g2 = gp[0] ** 2 + gp[1] ** 2 + gp[2] ** 2

        def em(x):  # exp(x) - 1 - x, by its series where that cancels
            return torch.where(x.abs() < 1e-2, x * x * (0.5 + x * (1 / 6 + x * (1 / 24 + x * (1 / 120 + x * (
                1 / 720 + x * (1 / 5040 + x / 40320)))))), torch.expm1(x) - x)
        rhs = (E - eb) + 0.5 * g2 + (E - eb) * p + E * em(p) - 1.5 * (
            (hc - pd) ** 2 * em(-2.0 * w) + 2.0 * w * (2.0 * hc * pd - pd * pd) + pd * pd) - 3.0 * hc * hc * c
        den = -self.k2 - (3.0 * hc * inv_dt + 6.0 * hc * hc + eb)
        if incr:  # the equation of the increment
            lap = sum(_shift(p, ax, 1) + _shift(p, ax, -1) for ax in range(3)) - 6.0 * p
            rhs = rhs - lap * float(n) ** 2 + (6.0 * hc * hc + eb) * p
        else:
            rhs = rhs - 3.0 * hc * inv_dt * p
        phi = torch.fft.irfftn(_ftn(rhs) / den, s=(n,) * 3)
        del rhs, g2, w
        e3 = torch.exp(3.0 * p)
        sig = []
        for s, (i, j) in enumerate(SYM):
            sig.append(_ftn(4.0 * e3 * kap * self.dep[4 + s] + 4.0 * gp[i] * gp[j] - 4.0 * (
                gp[i] * gc[j] + gc[i] * gp[j]) + 2.0 * gc[i] * gc[j]) * self.mask)
        del e3
        contr = sum((1.0 if i == j else 2.0) * self.kt[i] * self.kt[j] * sig[s] for s, (i, j) in enumerate(SYM))
        chi = torch.fft.irfftn(-0.75 / self.safe ** 2 * (contr - self.k2 * (sig[0] + sig[3] + sig[5]) / 3.0),
                               s=(n,) * 3)
        B = None
        if self.physics == "full" and elliptic:
            ef = torch.exp(p - c + 3.0 * p)
            S = [_ftn(ef * kap * self.dep[1 + i] - pd * (gp[i] - gc[i])) * self.mask for i in range(3)]
            kd = (self.kt[0] * S[0] + self.kt[1] * S[1] + self.kt[2] * S[2]) / self.safe
            B = [4.0 / self.safe * (S[i] - self.kt[i] * kd) for i in range(3)]
        return phi, chi, B, sig

    def solve(self, dtau):
        n = self.n
        real = lambda f: torch.fft.irfftn(f, s=(n,) * 3)  # noqa: E731
        if self.physics == "newtonian":
            self.phi = self.one_solve(None, None, None, 0.0, False, False)[0]
            return
        if dtau <= 0.0:
            phi, chi, _, _ = self.one_solve(None, None, None, 0.0, False, False)
            self.phi, self.chi, Bk, _ = self.one_solve(phi, chi, None, 0.0, False, True)
            self.delta, self.dtau_last = torch.zeros_like(self.phi), 0.0
            if self.physics == "full":
                self.B = [real(b) for b in Bk]
                self.a2b = [self.a_of(self.tau) ** 2 * b for b in Bk]
            return
        pd = self.delta / self.dtau_last if self.dtau_last > 0 else torch.zeros_like(self.phi)
        parabolic = bool(self.case.get("parabolic"))
        self.delta, self.chi, Bk, sig = self.one_solve(self.phi, self.chi, pd, 1.0 / dtau, True, not parabolic)
        self.phi = self.phi + self.delta
        self.dtau_last = dtau
        if self.physics == "full":  # h_ij acts on nothing and is not among the outputs
            if parabolic:
                kn = torch.sqrt(self.safe)
                kh = [k / kn for k in self.kt]
                at = {(i, j): s for s, (i, j) in enumerate(SYM)}
                v = [sum(sig[at[min(l, m), max(l, m)]] * kh[m] for m in range(3)) for l in range(3)]
                kv = kh[0] * v[0] + kh[1] * v[1] + kh[2] * v[2]
                am2 = self.a_of(self.tau - 0.5 * dtau) ** 2
                self.a2b = [(self.a2b[j] - 1j * dtau * am2 * (v[j] - kh[j] * kv) / kn) * self.mask for j in range(3)]
                Bk = [b / self.a_of(self.tau) ** 2 for b in self.a2b]
            self.B = [real(b) for b in Bk]

    def update(self, dtau, extra=None):
        a, ah = self.a_of(self.tau), self.a_of(self.tau + 0.5 * dtau)
        gphi = self.grad(self.phi)
        if extra is not None:
            gphi = [g + e for g, e in zip(gphi, extra)]
        new = []
        fields = [self.phi] + gphi
        if self.physics != "newtonian":
            fields += [self.chi] + self.grad(self.chi)
        if self.physics == "full":
            for b in self.B:
                fields += [b] + self.grad(b)
        for pos, u in self.sets:
            x1, u1 = torch.empty_like(pos), torch.empty_like(u)
            for b in range(0, pos.shape[0], CHUNK):
                sl = slice(b, min(b + CHUNK, pos.shape[0]))
                x, v = pos[sl], u[sl]
                g = [f for f in self.gather(fields, x)]
                if self.physics == "newtonian":
                    v = v - dtau * a * torch.stack(g[1:4], 1)
                    vel = v / ah
                else:
                    v2 = (v * v).sum(1)
                    e = torch.sqrt(a * a + v2)
                    force = [-(a * a + 2.0 * v2) / e * g[1 + d] + e * g[5 + d] for d in range(3)]
                    if self.physics == "full":
                        force = [force[d] - sum(v[:, j] * g[9 + 4 * j + d] for j in range(3)) for d in range(3)]
                    v = v + dtau * torch.stack(force, 1)
                    v2 = (v * v).sum(1, keepdim=True)
                    eh = torch.sqrt(ah * ah + v2)
                    vel = v / eh * (1.0 + (3.0 - v2 / (eh * eh)) * g[0][:, None] - g[4][:, None])
                    if self.physics == "full":
                        vel = vel + torch.stack([g[8], g[12], g[16]], 1)
                x = x + dtau * vel
                x = x - torch.floor(x)
                x1[sl] = torch.where(x >= 1.0, torch.zeros_like(x), x)
                u1[sl] = v
            new.append((x1, u1))
        self.sets = new
        self.tau += dtau

    def step(self, dtau, params=None):
        self.deposit()
        self.solve(self.last)
        extra = None
        if params is not None:
            acts, rms = self.features()
            extra = [rms * y for y in forward(params, acts)[0]]
        self.update(dtau, extra)
        self.last = dtau

    def features(self):
        g = self.grad(self.phi)
        rms = math.sqrt(float((g[0] ** 2 + g[1] ** 2 + g[2] ** 2).mean()))
        delta = self.dep[0] / self.dep[0].mean() - 1.0
        return torch.stack([torch.sign(delta) * torch.log1p(delta.abs())] + [x / rms for x in g]), rms


TAPS = [(dz, dy, dx) for dz in (-1, 0, 1) for dy in (-1, 0, 1) for dx in (-1, 0, 1)]


def _layers(params):
    o, out = 0, []
    for ci, co in LAYERS:
        w = params[o:o + co * ci * 27].double().reshape(co, ci, 27)
        o += co * ci * 27
        out.append((w, params[o:o + co].double()))
        o += co
    return out


def _roll3(x, d):
    return torch.roll(x, (-d[0], -d[1], -d[2]), dims=(1, 2, 3))


def _conv(x, w, b):
    """y[co](p) = b[co] + sum W[co][ci][t] x[ci](p + d_t); the channels are mixed before the shift."""
    y = b[:, None, None, None].expand((w.shape[0],) + x.shape[1:]).clone()
    flat = x.reshape(x.shape[0], -1)
    for t, d in enumerate(TAPS):
        y += _roll3((w[:, :, t].contiguous() @ flat).reshape((w.shape[0],) + x.shape[1:]), d)
    return y


def forward(params, x):
    (w1, b1), (w2, b2), (w3, b3) = _layers(params)
    a1 = _conv(x, w1, b1).clamp(min=0.0)
    a2 = _conv(a1, w2, b2).clamp(min=0.0)
    return _conv(a2, w3, b3), (x, a1, a2)


def backward(params, acts, dy):
    ls = _layers(params)
    out = []
    for li in (2, 1, 0):
        x, w = acts[li], ls[li][0]
        gw = torch.empty_like(w)
        dx = torch.zeros_like(x) if li else None
        for t, d in enumerate(TAPS):
            back = _roll3(dy, (-d[0], -d[1], -d[2])).reshape(dy.shape[0], -1)  # dy(p - d)
            gw[:, :, t] = back @ x.reshape(x.shape[0], -1).t().contiguous()
            if li:
                dx += (w[:, :, t].t().contiguous() @ back).reshape(x.shape)
        out.append(torch.cat([gw.reshape(-1), dy.sum(dim=(1, 2, 3))]))
        if li:
            dy = dx * (x > 0)
    return torch.cat(out[::-1])


def exact(case, seed):
    n, kind = case["n"], case["kind"]
    if kind == "fft":
        x = [f.double() for f in prepare(case, seed)["x"]]
        return {"k": [_ftn(f) for f in x], "x": x}
    pos, u = particles(case, seed)
    sets, masses = [(pos, u)], [1.0]
    if case.get("np2"):
        sets.append(second_species(case, seed))
        masses.append((0.1 / case["np2"]) / (0.9 / case["np"]))
    if kind == "train":
        target, m, v, perm, flip = training_rest(case, seed)
        pos, u, target = (t[:, perm].clone() for t in (pos, u, target))
        for d in range(3):
            if flip >> d & 1:
                pos[:, d] = 1.0 - pos[:, d]
                pos[:, d] -= (pos[:, d] >= 1.0).double()
                u[:, d], target[:, d] = -u[:, d], -target[:, d]
        sets = [(pos, u)]
    sim = Plain(case, sets, masses)
    if kind in ("evolve", "load"):
        dtau = case["dtau"] * sim.tau
        params = weights(seed) if case.get("closure") else None
        for _ in range(case["steps"] + (kind == "evolve")):
            sim.step(dtau, params)
        out = {"pos": sim.sets[0][0], "u": sim.sets[0][1], "phi": sim.phi}
        if case["physics"] != "newtonian":
            out["chi"] = sim.chi
        if case["physics"] == "full":
            out.update(zip(("bx", "by", "bz"), sim.B))
        return out
    if kind == "power":
        rho = sim.spread(pos, lambda sl: [torch.ones_like(pos[sl, 0])])[0]
        L = _box(case)
        half = torch.arange(n // 2 + 1, device="cuda", dtype=torch.float64)
        full = torch.fft.fftfreq(n, 1.0 / n, device="cuda", dtype=torch.float64)
        mx, my, mz = half[None, None, :], full[None, :, None], full[:, None, None]
        w = (torch.sinc(mx / n) * torch.sinc(my / n) * torch.sinc(mz / n)) ** 2
        p = (_ftn(rho).abs() / w) ** 2 * (L ** 3 / float(case["np"]) ** 2) - L ** 3 / case["np"]
        k = torch.sqrt(mx * mx + my * my + mz * mz)
        two = (torch.where((mx > 0) & (mx < n / 2), 2.0, 1.0) * torch.ones_like(k)).reshape(-1)
        b = torch.round(k).long().reshape(-1)
        size = int(b.max()) + 1
        modes, ps, ks = (torch.bincount(b, weights=x, minlength=size)[1:n // 2 + 1]
                         for x in (two, two * p.reshape(-1), two * k.reshape(-1)))
        return {"k": ks / modes * (2.0 * math.pi / L), "p": ps / modes, "modes": None}
    sim.deposit()
    sim.solve(0.0)
    if kind == "force":
        g = sim.grad(sim.phi)
        return {"g": torch.stack(sim.gather(g, sim.sets[0][0]), 1)}
    params = weights(seed)
    x, _ = sim.features()
    y, acts = forward(params, x)
    pred = torch.stack(sim.gather(list(y), pos), 1)
    r = pred - target.double()
    dpred = r * (2.0 / (3.0 * case["np"]))
    dy = sim.spread(pos, lambda sl: [dpred[sl, d] for d in range(3)])
    grad = backward(params, acts, dy)
    m = 0.9 * m.double() + 0.1 * grad
    v = 0.999 * v.double() + 0.001 * grad * grad
    c1, c2 = 1.0 - 0.9 ** 1000, 1.0 - 0.999 ** 1000
    params = params.double() - 1e-3 * (m / c1) / (torch.sqrt(v / c2) + 1e-8)
    return {"loss": float((r * r).mean()), "power": float((target.double() ** 2).mean()), "dpred": dpred, "grad": grad,
            "params": params, "m": m, "v": v}
