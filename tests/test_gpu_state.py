"""Checkpoint and restart through the C ABI (pm_get_state / pm_set_state).

* A run restarted in a fresh context from a checkpoint continues like the uninterrupted run
  (and, in FP64, like the oracle run over all steps): every part of the state (particles, phi of
  the two latest solves, chi, B, the tensor state and the parabolic a^2 B state) feeds the later
  steps, so a part left out shows up in the fields after the restart.
* The blob survives a restore byte for byte (host and device blobs are the same bytes).
* A checkpoint taken between pm_deposit and pm_solve_metric carries the deposit.
* Blobs of another configuration, truncated or with a damaged header are rejected.
* A sticky device error (non-finite phi set from the host, detected by the kick) is cleared by a
  restore, after which the run goes on as before.

Runs after a restore agree with the uninterrupted run to rounding, not bit for bit: particles
inside a cell are ordered by the sort's atomic counters.
"""
import numpy as np
import pytest

from oracle import pm as opm
from synth import config_particles
from tests.helpers import gpu_fields, oracle_fields, periodic_max_dx, rel_l2

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

TOL = {"fp64": (1e-11, 1e-10), "fp32": (1e-5, 1e-4)}  # (fields rel-L2, positions in mesh spacings)


def _say(msg):
    print(msg, flush=True)


def _ctx(n, n_p, box, physics, precision, b_route="elliptic"):
    from paper_2607_17929_amd import PMContext
    return PMContext(n, n_p, box, physics=physics, precision=precision, b_route=b_route)


def _state_of(ctx, physics):
    f = gpu_fields(ctx, physics)
    f["phi_prev"] = ctx.get_field("phi_prev").astype(np.float64)
    p, u = ctx.get_particles()
    return f, p, u.astype(np.float64), ctx.time()


CASES = [("fp64", "full", "parabolic"), ("fp64", "full", "elliptic"), ("fp64", "scalar", "elliptic"),
         ("fp32", "full", "parabolic"), ("fp64", "newtonian", "elliptic")]


@pytest.mark.parametrize("precision,physics,b_route", CASES)
def test_restart_continues_the_run(precision, physics, b_route):
    _say(f"restart {precision} {physics} {b_route}")
    pos, u, tau0, dtau = config_particles("zeldovich_32_scalar_fp64")
    n, box = 32, 320.0
    a = _ctx(n, pos.shape[0], box, physics, precision, b_route)
    u_in = u.astype(a.np_dtype)
    a.init_particles(pos, u_in, tau0)
    for _ in range(3):
        a.step(dtau)
    blob = a.get_state()
    for _ in range(4):
        a.step(dtau)
    ref = _state_of(a, physics)
    del a
    b = _ctx(n, pos.shape[0], box, physics, precision, b_route)
    b.set_state(blob)
    assert b.time()[2] == 3
    for _ in range(4):
        b.step(dtau)
    got = _state_of(b, physics)
    ftol, ptol = TOL[precision]
    assert got[3] == ref[3]  # tau, a and the step count
    for k in ref[0]:
        assert rel_l2(got[0][k], ref[0][k]) < ftol, (k, rel_l2(got[0][k], ref[0][k]))
    assert periodic_max_dx(got[1], ref[1], n) < ptol
    assert rel_l2(got[2], ref[2]) < ftol
    if precision == "fp64":
        # the restarted run against the oracle over all seven steps
        sim = opm.OracleSim(n=n, box_mpch=box, physics=physics, pos=pos, u=u, tau=tau0, b_route=b_route)
        for _ in range(7):
            sim.step(dtau)
        of = oracle_fields(sim, physics)
        for k in of:
            assert rel_l2(got[0][k], of[k]) < 1e-10, (k, rel_l2(got[0][k], of[k]))
        op, _ = sim.particles_by_id()
        assert periodic_max_dx(got[1], op, n) < 1e-9


def test_blob_round_trip_is_exact():
    _say("state blob round trip")
    pos, u, tau0, dtau = config_particles("zeldovich_32_scalar_fp64")
    a = _ctx(32, pos.shape[0], 320.0, "full", "fp32", "parabolic")
    a.init_particles(pos, u.astype(np.float32), tau0)
    for _ in range(2):
        a.step(dtau)
    host = a.get_state()
    dev = a.get_state(device=True)
    assert dev.numel() == host.size
    assert np.array_equal(dev.cpu().numpy(), host)
    b = _ctx(32, pos.shape[0], 320.0, "full", "fp32", "parabolic")
    b.set_state(dev)
    again = b.get_state()
    assert np.array_equal(again, host)
    # the restored context hands back the same fields and particles bit for bit
    for k in ("phi", "phi_prev", "chi", "bx", "hxy"):
        assert np.array_equal(a.get_field(k), b.get_field(k)), k
    pa, ua = a.get_particles()
    pb, ub = b.get_particles()
    assert np.array_equal(pa, pb) and np.array_equal(ua, ub)


def test_checkpoint_between_deposit_and_solve():
    _say("state between deposit and solve")
    pos, u, tau0, dtau = config_particles("zeldovich_32_scalar_fp64")
    a = _ctx(32, pos.shape[0], 320.0, "full", "fp64")
    a.init_particles(pos, u, tau0)
    a.step(dtau)
    after_step = a.get_state().size
    a.deposit()
    blob = a.get_state()
    assert blob.size >= after_step + 10 * 32 ** 3 * 8  # the ten deposit components travel with it
    b = _ctx(32, pos.shape[0], 320.0, "full", "fp64")
    b.set_state(blob)
    for c in (a, b):
        c.solve_metric(dtau)
        c.update_particles(dtau)
    fa, fb = gpu_fields(a, "full"), gpu_fields(b, "full")
    for k in fa:
        assert rel_l2(fb[k], fa[k]) < 1e-12, k
    from paper_2607_17929_amd import PMError
    with pytest.raises(PMError):
        _ctx(32, pos.shape[0], 320.0, "full", "fp64").solve_metric(dtau)  # no state, no deposit


def test_foreign_or_damaged_blobs_are_rejected():
    from paper_2607_17929_amd import PMError
    _say("state blob validation")
    pos, u, tau0, dtau = config_particles("zeldovich_32_scalar_fp64")
    a = _ctx(32, pos.shape[0], 320.0, "scalar", "fp64")
    a.init_particles(pos, u, tau0)
    a.step(dtau)
    blob = a.get_state()
    for other in (_ctx(32, pos.shape[0], 320.0, "scalar", "fp32"), _ctx(32, pos.shape[0], 320.0, "full", "fp64"),
                  _ctx(16, pos.shape[0], 320.0, "scalar", "fp64"), _ctx(32, pos.shape[0] - 1, 320.0, "scalar", "fp64")):
        with pytest.raises(PMError) as e:
            other.set_state(blob)
        assert e.value.status == -1
    with pytest.raises(PMError):
        a.set_state(blob[: blob.size // 2])
    bad = blob.copy()
    bad[0] ^= 0xFF
    with pytest.raises(PMError):
        a.set_state(bad)
    bad = blob.copy()
    bad[112:120] = 0xFF  # the first section's offset
    with pytest.raises(PMError):
        a.set_state(bad)
    # the context still holds its own state and steps on
    a.step(dtau)
    assert a.time()[2] == 2


def test_restore_clears_a_sticky_device_error():
    from paper_2607_17929_amd import PMError
    _say("state restore after a device error")
    pos, u, tau0, dtau = config_particles("zeldovich_32_scalar_fp64")
    a = _ctx(32, pos.shape[0], 320.0, "scalar", "fp64")
    a.init_particles(pos, u, tau0)
    for _ in range(2):
        a.step(dtau)
    blob = a.get_state()
    ref = _ctx(32, pos.shape[0], 320.0, "scalar", "fp64")
    ref.set_state(blob)
    ref.step(dtau)
    bad = np.full((32, 32, 32), np.nan)
    a.set_field("phi", bad)
    a.update_particles(dtau)  # non-finite kick: the kernel flags it and parks the particles
    with pytest.raises(PMError) as e:
        a.sync()
    assert e.value.status == -4
    with pytest.raises(PMError):
        a.step(dtau)  # sticky
    a.set_state(blob)
    a.step(dtau)
    fa, fr = gpu_fields(a, "scalar"), gpu_fields(ref, "scalar")
    for k in fa:
        assert rel_l2(fa[k], fr[k]) < 1e-12, k
    pa, _ = a.get_particles()
    pr, _ = ref.get_particles()
    assert periodic_max_dx(pa, pr, 32) < 1e-10


def _header_sections(blob):
    """(offset, bytes) of each section of a state blob, read from its header (magic, version,
    section count, configuration, times, flags, total, then 32 offsets and 32 sizes as uint64)."""
    nsec = int(np.frombuffer(blob[12:16].tobytes(), dtype=np.uint32)[0])
    off = np.frombuffer(blob[112:112 + 8 * 32].tobytes(), dtype=np.uint64)[:nsec]
    size = np.frombuffer(blob[368:368 + 8 * 32].tobytes(), dtype=np.uint64)[:nsec]
    return [(int(o), int(b)) for o, b in zip(off, size)]


def test_damaged_blob_bodies_are_rejected():
    """The body of a checkpoint is checked on the device before the context runs on it: cell offsets
    that do not end at the particle count or decrease, a position outside [0, 1), a particle moved
    into another cell's range and an identifier out of range each give PM_EINVAL; the context then
    holds no particles (the next deposit is out of order) until a good blob is restored."""
    from paper_2607_17929_amd import PMError
    _say("state blob body validation")
    pos, u, tau0, dtau = config_particles("zeldovich_32_scalar_fp64")
    n, n_p = 32, pos.shape[0]
    a = _ctx(n, n_p, 320.0, "scalar", "fp64")
    a.init_particles(pos, u, tau0)
    a.step(dtau)
    blob = a.get_state()
    sec = _header_sections(blob)
    (o_pos, _), (o_mom, _), (o_id, _), (o_cs, b_cs) = sec[:4]
    assert b_cs == (n ** 3 + 1) * 4
    cs = np.frombuffer(blob[o_cs:o_cs + b_cs].tobytes(), dtype=np.uint32).copy()
    px = np.frombuffer(blob[o_pos:o_pos + 8 * n_p].tobytes(), dtype=np.float64).copy()

    def with_cs(c):
        b = blob.copy()
        b[o_cs:o_cs + b_cs] = np.frombuffer(c.astype(np.uint32).tobytes(), dtype=np.uint8)
        return b

    def with_x(i, x):
        b = blob.copy()
        b[o_pos + 8 * i:o_pos + 8 * i + 8] = np.frombuffer(np.float64(x).tobytes(), dtype=np.uint8)
        return b

    damaged = {}
    c = cs.copy(); c[-1] = n_p + 1; damaged["total"] = with_cs(c)
    c = cs.copy(); k = int(np.argmax(np.diff(cs) > 0)); c[k + 1] = c[k] - 1 if c[k] > 0 else c[k + 2] + 5
    damaged["decreasing"] = with_cs(c)
    damaged["outside"] = with_x(0, 1.5)
    damaged["nan"] = with_x(1, float("nan"))
    damaged["other cell"] = with_x(2, (px[2] + 0.5) % 1.0)
    b = blob.copy(); b[o_id:o_id + 4] = np.frombuffer(np.uint32(n_p).tobytes(), dtype=np.uint8)
    damaged["identifier"] = b
    target = _ctx(n, n_p, 320.0, "scalar", "fp64")
    for name, bad in damaged.items():
        _say(f"  damaged body: {name}")
        with pytest.raises(PMError) as e:
            target.set_state(bad)
        assert e.value.status == -1, name
        with pytest.raises(PMError) as e:
            target.deposit()
        assert e.value.status == -5, name
    target.set_state(blob)
    target.step(dtau)
    a.step(dtau)
    fa, ft = gpu_fields(a, "scalar"), gpu_fields(target, "scalar")
    for k in fa:
        assert rel_l2(ft[k], fa[k]) < 1e-12, k


DET_CASES = [("fp32", "full", "elliptic", "zeldovich_32"), ("fp32", "full", "parabolic", "clustered_64"),
             ("fp64", "scalar", "elliptic", "zeldovich_32")]


def _det_inputs(kind):
    if kind == "zeldovich_32":
        pos, u, tau0, dtau = config_particles("zeldovich_32_scalar_fp64")
        return 32, 320.0, pos, u, tau0, dtau
    # many particles per cell: most of the sums over a cell have several terms
    r = np.random.default_rng(61)
    n = 64
    centers = r.random((6, 3))
    pos = (centers[r.integers(0, 6, 60000)] + 0.8 / n * r.standard_normal((60000, 3))) % 1.0
    u = 2e-3 * r.standard_normal((60000, 3))
    tau0 = opm.Background(640.0).tau(0.2)
    return n, 640.0, pos, u, tau0, 0.01 * tau0


def _det_state(ctx, physics):
    f = {k: v.copy() for k, v in gpu_fields(ctx, physics).items()}
    p, u = ctx.get_particles()
    return f, p, u


@pytest.mark.parametrize("precision,physics,b_route,kind", DET_CASES)
def test_deterministic_runs_and_restart_are_bitwise_equal(precision, physics, b_route, kind):
    """With PM_FLAG_DETERMINISTIC two runs from the same inputs give bitwise identical fields and
    particles after ten steps, and so does a run restarted from a checkpoint taken after five steps in
    a fresh context (the checkpoint holds the store in its deterministic order)."""
    from paper_2607_17929_amd import PMContext
    _say(f"deterministic {precision} {physics} {b_route} {kind}")
    n, box, pos, u, tau0, dtau = _det_inputs(kind)
    runs = []
    blob = None
    for k in range(2):
        ctx = PMContext(n, pos.shape[0], box, physics=physics, precision=precision, b_route=b_route,
                        deterministic=True)
        ctx.init_particles(pos, u.astype(ctx.np_dtype), tau0)
        for s in range(10):
            ctx.step(dtau)
            if k == 0 and s == 4:
                blob = ctx.get_state()
        runs.append(_det_state(ctx, physics))
        del ctx
    ctx = PMContext(n, pos.shape[0], box, physics=physics, precision=precision, b_route=b_route, deterministic=True)
    ctx.set_state(blob)
    for _ in range(5):
        ctx.step(dtau)
    runs.append(_det_state(ctx, physics))
    ref = runs[0]
    for other in runs[1:]:
        for name in ref[0]:
            assert np.array_equal(other[0][name], ref[0][name]), name
        assert np.array_equal(other[1], ref[1]) and np.array_equal(other[2], ref[2])
    # the same as an ordinary run up to rounding
    ctx = PMContext(n, pos.shape[0], box, physics=physics, precision=precision, b_route=b_route)
    ctx.init_particles(pos, u.astype(ctx.np_dtype), tau0)
    for _ in range(10):
        ctx.step(dtau)
    plain = _det_state(ctx, physics)
    tol = 1e-10 if precision == "fp64" else 1e-5
    for name in ref[0]:
        assert rel_l2(plain[0][name], ref[0][name]) < tol, name
    assert periodic_max_dx(plain[1], ref[1], n) < (1e-9 if precision == "fp64" else 1e-4)


@pytest.mark.parametrize("precision", ["fp32", "fp64"])
def test_blob_holds_the_particles_as_separate_arrays(precision):
    """The sections of the particles are x | y | z, u_x | u_y | u_z (1280 bytes after each of the first two arrays)
    and the identifiers, in the order of the cells, whatever records the store itself keeps; the same bytes are
    restored.  Odd counts, so that no array ends on a vector boundary; exact (bytes are moved, not computed)."""
    from paper_2607_17929_amd import PMContext
    _say(f"blob layout {precision}")
    n, n1, n2, gap = 16, 1001, 333, 1280
    rng = np.random.default_rng(5)
    ctx = PMContext(n, n1, 100.0, physics="newtonian", precision=precision, n_particles_2=n2, mass_fraction_2=0.25)
    sets = []
    for m in (n1, n2):
        sets.append((rng.random((m, 3)), (1e-3 * rng.standard_normal((m, 3))).astype(ctx.np_dtype)))
    ctx.init_particles(*sets[0], 0.1)
    ctx.init_particles_2(*sets[1])
    ctx.step(1e-3)
    blob = ctx.get_state()
    head = blob[:1024].view(np.uint64)
    off = head[14:46].astype(np.int64)  # after 112 bytes of scalars
    rs = np.dtype(ctx.np_dtype).itemsize
    for k, (m, get) in enumerate(((n1, ctx.get_particles), (n2, ctx.get_particles_2))):
        o_pos, o_mom, o_id = off[4 * k:4 * k + 3]
        ids = blob[o_id:o_id + 4 * m].view(np.uint32)
        assert np.array_equal(np.sort(ids), np.arange(m))
        pos, u = get()
        cell = np.floor(pos[ids] * n).astype(np.int64)
        key = (cell[:, 2] * n + cell[:, 1]) * n + cell[:, 0]
        assert (np.diff(key) >= 0).all()
        for d in range(3):
            x = o_pos + d * (8 * m + gap)
            v = o_mom + d * (rs * m + gap)
            assert np.array_equal(blob[x:x + 8 * m].view(np.float64), pos[ids, d])
            assert np.array_equal(blob[v:v + rs * m].view(ctx.np_dtype), u[ids, d])
            if d < 2:
                assert not blob[x + 8 * m:x + 8 * m + gap].any() and not blob[v + rs * m:v + rs * m + gap].any()
    again = PMContext(n, n1, 100.0, physics="newtonian", precision=precision, n_particles_2=n2, mass_fraction_2=0.25)
    again.set_state(blob)
    assert np.array_equal(again.get_state(), blob)
