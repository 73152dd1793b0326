"""Branches that only meshes of 128^3 and more reach."""
import numpy as np
import pytest

from synth import config_particles
from tests.test_gpu_parity import FIELD_TOL, POS_TOL, _run_both

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("n", [128, 256])
def test_fp64_scalar_narrow_fourier_tiles(n):
    """The Fourier-space kernel where its tiles are narrower than the 4 kx that an FP64 scalar row wants: 2 kx at 128^3,
    1 kx at 256^3; 32^3 particles, two steps and one."""
    print("fp64 scalar", n, flush=True)
    pos, u, tau0, dtau = config_particles("zeldovich_32_scalar_fp64")
    worst, dxmax, urel, *_ = _run_both(n, 320.0, "scalar", "fp64", pos, u, tau0, [dtau] * (256 // n))
    print(worst, dxmax, urel, flush=True)
    for k, v in worst.items():
        assert v < FIELD_TOL["fp64"], (k, v)
    assert dxmax < POS_TOL["fp64"]


@pytest.mark.parametrize("n", [128, 512])
def test_power_spectrum_mode_counts(n):
    """The number of modes of every shell, exactly: |m|^2 is an integer and no shell's edge is one."""
    from paper_2607_17929_amd import PMContext
    print("mode counts", n, flush=True)
    ctx = PMContext(n, 1001, 100.0, physics="newtonian", precision="fp32")
    ctx.init_particles(np.random.default_rng(6).random((1001, 3)), np.zeros((1001, 3), np.float32), 1.0)
    _, _, modes = ctx.power_spectrum()
    h = n // 2
    m = np.arange(h + 1, dtype=np.int64)
    times = np.where((m > 0) & (m < h), 2, 1)  # m and -m
    want = np.zeros(h + 1, np.int64)
    yz, w_yz = (m[:, None] ** 2 + m[None, :] ** 2).reshape(-1), np.outer(times, times).reshape(-1)
    for kx in range(h + 1):
        b = np.rint(np.sqrt((yz + kx * kx).astype(np.float64))).astype(np.int64)
        want += np.bincount(b, weights=w_yz * times[kx], minlength=h + 1)[:h + 1].astype(np.int64)
    assert np.array_equal(modes, want[1:])


@pytest.mark.parametrize("precision,n", [("fp64", 256), ("fp32", 512)])
def test_fft_dense_rows_of_large_meshes(precision, n):
    """Every mode and value of a transform there and back where the z pass takes its tiles in XCD order (256^3 and more,
    the last tile one column wide), against torch's FP64 transform; bars of the small meshes' FFT test."""
    from paper_2607_17929_amd import PMContext
    print("fft", precision, n, flush=True)
    ctx = PMContext(n, 8, 100.0, physics="newtonian", precision=precision)
    f = torch.randn((n, n, n), dtype=ctx.dtype, device="cuda", generator=torch.Generator("cuda").manual_seed(n))
    fk = ctx.debug_fft(f, 1)
    ref = torch.fft.rfftn(f.double())
    tol = (1e-13 if precision == "fp64" else 3e-7) * np.log2(n)
    assert float((fk.to(ref.dtype) - ref).norm() / ref.norm()) < tol
    back = ctx.debug_fft(fk, -1)
    assert float((back.double() - f.double()).norm() / f.double().norm()) < tol
