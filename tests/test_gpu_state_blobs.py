"""Device checkpoints at any address: aligned ones are unpacked and packed in place, others by way of a copy; the bytes
and the restored state are the same."""
import ctypes as C

import numpy as np
import pytest

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("shift", [0, 8, 4, 1])
@pytest.mark.parametrize("precision", ["fp32", "fp64"])
def test_device_blob_at_any_alignment(precision, shift):
    """Two species of odd counts; exact (bytes are moved, not computed)."""
    from paper_2607_17929_amd import PMContext
    print("device blob", precision, shift, flush=True)
    n, n1, n2 = 16, 1001, 333
    rng = np.random.default_rng(8)
    make = lambda: PMContext(n, n1, 100.0, physics="newtonian", precision=precision, n_particles_2=n2,  # noqa: E731
                             mass_fraction_2=0.25)
    a, b = make(), make()
    a.init_particles(rng.random((n1, 3)), (1e-3 * rng.standard_normal((n1, 3))).astype(a.np_dtype), 0.1)
    a.init_particles_2(rng.random((n2, 3)), (1e-3 * rng.standard_normal((n2, 3))).astype(a.np_dtype))
    a.step(1e-3)
    host = a.get_state()
    room = torch.full((host.size + 16,), 0x5a, dtype=torch.uint8, device="cuda")
    size = C.c_size_t(host.size)
    assert a.lib.pm_get_state(a.ctx, C.c_void_p(room.data_ptr() + shift), C.byref(size), 1) == 0
    assert size.value == host.size
    got = room.cpu().numpy()
    assert np.array_equal(got[shift:shift + host.size], host)
    assert np.all(got[:shift] == 0x5a) and np.all(got[shift + host.size:] == 0x5a)
    assert b.lib.pm_set_state(b.ctx, C.c_void_p(room.data_ptr() + shift), host.size, 1) == 0
    assert np.array_equal(b.get_state(), host)
    for x, y in zip(a.get_particles() + a.get_particles_2(), b.get_particles() + b.get_particles_2()):
        assert np.array_equal(x, y)
