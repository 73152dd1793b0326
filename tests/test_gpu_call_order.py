"""Calls that go through the particle store's cell offsets are refused while the context holds no particles."""
import numpy as np
import pytest

from oracle import cnn

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

N, NP, ESTATE = 16, 999, -5


def _ctx(**kw):
    from paper_2607_17929_amd import PMContext
    return PMContext(N, NP, 100.0, physics="scalar", precision="fp32", closure=True, **kw)


def _load(ctx, seed=1):
    rng = np.random.default_rng(seed)
    ctx.init_particles(rng.random((NP, 3)), np.zeros((NP, 3), np.float32), 12.0)


def _forward(ctx):
    ctx.deposit()
    ctx.solve_metric(0.0)
    ctx.closure_set_params(torch.zeros(cnn.N_PARAMS))
    ctx.closure_forward(False)


def _refused(call, *args):
    from paper_2607_17929_amd import PMError
    with pytest.raises(PMError) as e:
        call(*args)
    assert e.value.status == ESTATE, call.__name__


def _closure_calls_refused(ctx):
    v = torch.zeros((NP, 3), device="cuda")
    _refused(ctx.closure_gather)
    _refused(ctx.closure_loss, v)
    _refused(ctx.closure_backward, v)


def test_no_particles_after_a_damaged_checkpoint():
    """A forward pass, then a restore whose body is refused: its cell offsets are in the workspace, so everything that reads
    them gives PM_ESTATE (on the host, before a launch), also after phi was set; a good blob makes it all work again."""
    from paper_2607_17929_amd import PMError
    print("calls after a damaged checkpoint", flush=True)
    ctx = _ctx()
    _load(ctx)
    blob = ctx.get_state()
    _forward(ctx)
    bad = blob.copy()
    off = np.frombuffer(blob[112:112 + 8 * 4].tobytes(), np.uint64)[3]  # the fourth section: cell offsets
    bad[int(off):int(off) + 4 * (N ** 3 + 1)] = 0xff
    with pytest.raises(PMError) as e:
        ctx.set_state(bad)
    assert e.value.status == -1
    _closure_calls_refused(ctx)
    _refused(ctx.update_particles, 0.01)
    ctx.set_field("phi", np.zeros((N, N, N), np.float32))
    _refused(ctx.update_particles, 0.01)
    _refused(ctx.gather_grad_phi)
    _refused(ctx.power_spectrum)
    ctx.closure_forward(False)
    _closure_calls_refused(ctx)
    ctx.set_state(blob)
    _forward(ctx)
    assert ctx.closure_gather().shape == (NP, 3)
    ctx.update_particles(0.01)


def test_update_needs_both_species():
    """phi set by the caller stands for a solve, but not for particles of either species."""
    print("update without particles", flush=True)
    ctx = _ctx(n_particles_2=77, mass_fraction_2=0.1)
    ctx.set_field("phi", np.zeros((N, N, N), np.float32))
    _refused(ctx.update_particles, 0.01)
    _load(ctx)
    ctx.set_field("phi", np.zeros((N, N, N), np.float32))
    _refused(ctx.update_particles, 0.01)
    ctx.init_particles_2(np.random.default_rng(3).random((77, 3)), np.zeros((77, 3), np.float32))
    ctx.set_field("phi", np.zeros((N, N, N), np.float32))
    ctx.update_particles(0.01)


def test_forward_pass_ends_with_a_new_load():
    """After particles are loaded anew the former set's network output and activations count no longer."""
    print("closure calls after a reload", flush=True)
    ctx = _ctx()
    _load(ctx)
    _forward(ctx)
    assert ctx.closure_gather().shape == (NP, 3)
    _load(ctx, 2)
    _closure_calls_refused(ctx)
    _forward(ctx)
    assert ctx.closure_gather().shape == (NP, 3)
