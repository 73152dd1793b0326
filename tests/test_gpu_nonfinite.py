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
