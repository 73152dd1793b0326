"""Roundings that a run's last bits hang on, against NumPy with every rounding written out (a fused multiply-add is formed
in FP64: the product of two FP32 values is exact there)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

F = np.float32


def _fma(a, b, c):
    return (np.asarray(a, np.float64) * np.asarray(b, np.float64) + np.asarray(c, np.float64)).astype(F)


def _rsq(x):
    """The FP32 values that an instruction accurate to one unit in the last place may give for 1 / sqrt(x)."""
    r = (1.0 / np.sqrt(x.astype(np.float64))).astype(F)
    return [np.nextafter(r, F(0)), r, np.nextafter(r, F(np.inf))]


@pytest.mark.parametrize("physics", ["scalar", "full"])
def test_kick_of_hot_particles_fp32(physics):
    """One hot particle on every vertex of a 16^3 mesh, so that the gathered fields and gradients are the vertex's own,
    in given phi and chi.  The squares are summed as fma(u_z, u_z, fma(u_y, u_y, u_x u_x)) before the kick and as
    fma(u_z, u_z, fma(u_x, u_x, u_y u_y)) after it.  Momenta: equal but for two in a million (the FP64 sums in _fma are
    rounded twice); positions: to 1e-14, where a last bit of the FP32 velocity is 1e-9."""
    from paper_2607_17929_amd import PMContext
    from paper_2607_17929_amd.pm import background
    print("kick rounding", physics, flush=True)
    n, box, tau, dtau = 16, 100.0, 12.0, 0.05
    rng = np.random.default_rng(3)
    ctx = PMContext(n, n ** 3, box, physics=physics, precision="fp32")
    z, y, x = np.meshgrid(*[np.arange(n)] * 3, indexing="ij")
    pos = np.stack([x, y, z], -1).reshape(-1, 3) / n
    a, ah = F(background(box, tau)[0]), F(background(box, tau + 0.5 * dtau)[0])
    u = (rng.standard_normal((n ** 3, 3)) * a).astype(F)
    phi, chi = (0.3 * rng.standard_normal((2, n, n, n))).astype(F)
    ctx.init_particles(pos, u, tau)
    ctx.set_field("phi", phi)
    ctx.set_field("chi", chi)
    ctx.update_particles(dtau)
    gpos, gu = ctx.get_particles()

    def grad(f):
        return [((np.roll(f, -1, ax) - np.roll(f, 1, ax)) * F(0.5 * n)).reshape(-1) for ax in (2, 1, 0)]

    gp, gc, p, c = grad(phi), grad(chi), phi.reshape(-1), chi.reshape(-1)
    ux, uy, uz = u.T
    u2 = _fma(uz, uz, _fma(uy, uy, ux * ux))
    e2 = a * a + u2
    kick = drift = np.zeros(n ** 3, bool)
    for ie in _rsq(e2):
        cphi, e = -(a * a + F(2) * u2) * ie, e2 * ie
        v = np.stack([_fma(F(dtau), _fma(cphi, gp[d], e * gc[d]), u[:, d]) for d in range(3)], -1)
        kick = kick | (v == gu).all(1)
    vx, vy, vz = gu.T
    v2 = _fma(vz, vz, _fma(vx, vx, vy * vy))
    for ieh in _rsq(ah * ah + v2):
        fac = (_fma(_fma(-(v2 * ieh), ieh, 3.0), p, 1.0) - c) * ieh
        d = gpos - (pos + dtau * (gu * fac[:, None]).astype(np.float64))
        drift = drift | (np.abs(d - np.rint(d)).max(1) < 1e-14)
    assert np.mean(~kick) <= 2e-6 and np.mean(~drift) <= 2e-6, (np.mean(~kick), np.mean(~drift))


def test_deposit_fp32_stresses_are_running_sums():
    """FP32 sums of the stresses in the order of the store: through the planes of cells, the cells in row-major order and
    (deterministic mode) the particles of a cell by identifier, each term added with one rounding.  Cells of 60, 13, 700
    and 5 particles next to each other; all have the same momentum, and one that sits on a vertex far off gives the
    term itself, with weight one.  Equal but for one value in a thousand (_fma is rounded twice: 1e-9 a term)."""
    from paper_2607_17929_amd import PMContext
    print("deposit running sums", flush=True)
    n = 16
    rng = np.random.default_rng(9)
    cells = {(4, 5, 6): 60, (5, 5, 6): 13, (4, 6, 6): 700, (5, 6, 7): 5, (5, 5, 7): 41}
    pos = [(np.array(c) + rng.random((k, 3))) / n for c, k in cells.items()] + [np.full((1, 3), 12 / n)]
    pos = np.concatenate(pos)
    u = np.tile(np.array([0.11, -0.07, 0.05], F), (pos.shape[0], 1))
    ctx = PMContext(n, pos.shape[0], 100.0, physics="scalar", precision="fp32", deterministic=True)
    ctx.init_particles(pos, u, 12.0)
    ctx.deposit()
    s = pos * n
    cell = np.floor(s).astype(int)
    f = (s - cell).astype(F)
    order = np.lexsort((np.arange(len(pos)), cell[:, 0], cell[:, 1], cell[:, 2]))
    wrong = total = 0
    for name in ("nxx", "nxy", "nxz", "nyy", "nyz", "nzz"):
        got = ctx.get_field(name)
        t = got[12, 12, 12]
        want = np.zeros_like(got)
        want[12, 12, 12] = t
        for i in order[cell[order, 0] != 12]:
            for dy in (0, 1):
                for dx in (0, 1):
                    wx, wy = f[i, 0] if dx else F(1) - f[i, 0], f[i, 1] if dy else F(1) - f[i, 1]
                    wh = wx * wy * f[i, 2]
                    for dz, wz in ((1, wh), (0, _fma(wx, wy, -wh))):
                        at = (cell[i, 2] + dz, cell[i, 1] + dy, cell[i, 0] + dx)
                        want[at] = _fma(wz, t, want[at])
        wrong += np.sum(got != want)
        total += np.sum(want != 0)
    assert total > 100 and wrong <= 1e-3 * total, (wrong, total)


def test_two_species_deterministic_run_repeats():
    """Full physics, parabolic B, a hot second species, clustered cells among them: two runs of five steps, in contexts of
    their own, are equal to the bit."""
    from paper_2607_17929_amd import PMContext
    print("two species, deterministic", flush=True)
    n, n1, n2, tau = 32, 30011, 5003, 10.0
    rng = np.random.default_rng(12)
    pos = np.concatenate([rng.random((n1 - 4000, 3)), (0.3 + 0.02 * rng.standard_normal((4000, 3))) % 1.0])
    u = (1e-4 * rng.standard_normal((n1, 3))).astype(F)
    pos2, u2 = rng.random((n2, 3)), (0.2 * rng.standard_normal((n2, 3))).astype(F)
    runs = []
    for _ in range(2):
        ctx = PMContext(n, n1, 128.0, physics="full", precision="fp32", b_route="parabolic", n_particles_2=n2,
                        mass_fraction_2=0.1, deterministic=True)
        ctx.init_particles(pos, u, tau)
        ctx.init_particles_2(pos2, u2)
        for _ in range(5):
            ctx.step(0.01 * tau)
        runs.append([*ctx.get_particles(), *ctx.get_particles_2(), *(ctx.get_field(f) for f in ("phi", "chi", "bx", "hxy"))])
    for a, b in zip(*runs):
        assert np.array_equal(a, b)
