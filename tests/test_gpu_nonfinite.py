"""Infinities go through the kernels that pad their products: padding counts as zero, never as zero times a value."""
import numpy as np
import pytest

from oracle import cnn

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def test_closure_forward_infinite_activations():
    """Biases that bfloat16 rounds to infinity make every activation of the first layer infinite; with weights of one the
    second layer and the output are infinite too (the convolution's 28th tap is padding)."""
    from paper_2607_17929_amd import PMContext
    print("closure, infinite activations", flush=True)
    n, np1 = 16, 4096
    rng = np.random.default_rng(2)
    ctx = PMContext(n, np1, 100.0, physics="scalar", precision="fp32", closure=True)
    ctx.init_particles(rng.random((np1, 3)), np.zeros((np1, 3), np.float32), 12.0)
    ctx.deposit()
    ctx.solve_metric(0.0)
    params = np.zeros(cnn.N_PARAMS, np.float32)
    first = 16 * 4 * 27
    params[first:first + 16] = 3.4e38
    second = first + 16 + 16 * 16 * 27
    params[first + 16:second] = 1.0
    params[second + 16:-3] = 1.0
    ctx.closure_set_params(torch.tensor(params))
    ctx.closure_forward(False)
    out = ctx.closure_gather().cpu().numpy()
    assert np.all(out == np.inf), (np.mean(out == np.inf), out[:2])


def _cell_of_13(n=16):
    """A cell of 13 particles (not a multiple of the four that one matrix product takes), the last one by identifier
    being the set's last, in a thin background."""
    rng = np.random.default_rng(4)
    pos = np.concatenate([rng.random((n * n, 3)), (np.array([9, 6, 3]) + 0.1 + 0.8 * rng.random((13, 3))) / n])
    return pos[np.any(np.floor(pos * n) != [9, 6, 3], axis=1) | (np.arange(len(pos)) >= n * n)]


def test_deposit_fp64_infinite_energy():
    """A momentum whose square overflows: n00 is infinite on the particle's 8 vertices and finite elsewhere, n0x is
    finite everywhere."""
    from paper_2607_17929_amd import PMContext
    print("deposit, infinite energy", flush=True)
    pos = _cell_of_13()
    u = np.full(pos.shape, 1e-3)
    u[-1, 0] = 1e200
    ctx = PMContext(16, pos.shape[0], 100.0, physics="scalar", precision="fp64", deterministic=True)
    ctx.init_particles(pos, u, 12.0)
    ctx.deposit()
    want = np.zeros((16, 16, 16), bool)
    want[3:5, 6:8, 9:11] = True
    n00, n0x = ctx.get_field("n00"), ctx.get_field("n0x")
    assert np.array_equal(n00 == np.inf, want) and np.isfinite(n00[~want]).all()
    assert np.isfinite(n0x).all() and np.array_equal(n0x > 1e150, want)


@pytest.mark.parametrize("precision", ["fp32", "fp64"])
def test_closure_backward_infinite_residual(precision):
    """An infinite residual of one particle: the output bias's gradient of that component is infinite, the others' are
    finite."""
    from paper_2607_17929_amd import PMContext
    print("closure backward, infinite residual", precision, flush=True)
    pos = _cell_of_13()
    ctx = PMContext(16, pos.shape[0], 100.0, physics="scalar", precision=precision, closure=True, deterministic=True)
    ctx.init_particles(pos, np.zeros(pos.shape, ctx.np_dtype), 12.0)
    ctx.deposit()
    ctx.solve_metric(0.0)
    ctx.closure_set_params(torch.tensor(np.random.default_rng(5).standard_normal(cnn.N_PARAMS), dtype=torch.float32))
    ctx.closure_forward(False)
    dpred = torch.ones(pos.shape, dtype=torch.float32)
    dpred[-1, 0] = np.inf
    bias = ctx.closure_backward(dpred).cpu().numpy()[-3:]
    assert bias[0] == np.inf and np.isfinite(bias[1:]).all(), bias
