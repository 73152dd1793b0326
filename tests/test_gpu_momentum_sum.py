"""The total momentum at counts around the edges of its sum: one particle, less than a wave, a workgroup's share, a
remainder of one, more blocks than partials are kept for."""
import math

import numpy as np
import pytest

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("precision", ["fp32", "fp64"])
@pytest.mark.parametrize("count", [1, 63, 1024, 1025, 320 * 1024, 320 * 1024 + 1, 1000003])
def test_total_momentum(count, precision):
    """Against the exactly rounded sum, to 1e-13 of the sum of magnitudes (a million terms in FP64, summed in chains of
    at most 13 and trees)."""
    from paper_2607_17929_amd import PMContext
    print("momentum", count, precision, flush=True)
    rng = np.random.default_rng(count)
    ctx = PMContext(16, count, 100.0, physics="newtonian", precision=precision)
    u = (1e-3 * rng.standard_normal((count, 3))).astype(ctx.np_dtype)
    ctx.init_particles(rng.random((count, 3)), u, 1.0)
    got = ctx.diagnostics()["momentum"]
    for d in range(3):
        v = u[:, d].astype(np.float64)
        assert abs(got[d] - math.fsum(v)) <= 1e-13 * np.abs(v).sum()
