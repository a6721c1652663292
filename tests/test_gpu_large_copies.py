"""Fields and checkpoints of 8 MiB and more leave the device through a ring of
pinned 1 MiB chunks and worker threads; smaller ones, and pinned destinations,
in one copy. Right after vklb_init in the delta basis the fields are the
initial ones, value for value."""
import ctypes

import numpy as np
import pytest

from paper_2608_04283_amd import inputs as I

pytestmark = pytest.mark.gpu

MI = 1 << 17  # doubles of 1 MiB


def linear(n):
    P = I.Problem(name="linear", system="linear", dim=1, n=(n,), bc=("periodic", "periodic"), max_steps=8)
    return P.with_(U0=np.random.default_rng(n).uniform(0.5, 1.5, (1, n)))


@pytest.mark.parametrize("n", [8 * MI - 1, 8 * MI, 8 * MI + 1, 9 * MI, 16 * MI, 16 * MI + 77, 41 * MI - 3])
def test_moments_are_the_initial_fields(gpu, n):
    import torch
    P = linear(n)
    s = gpu.Solver(P, precision="fp64", basis=2)
    for k in range(3):
        s.init(P.U0 * (k + 1))
        U, t, steps = s.moments()
        assert t == 0.0 and steps == 0 and np.array_equal(U, P.U0 * (k + 1))
    pinned = torch.empty((1, n), dtype=torch.float64, pin_memory=True).numpy()
    s._check(gpu.lib().vklb_moments(s._h, pinned.ctypes.data_as(ctypes.POINTER(ctypes.c_double)), None, None))
    assert np.array_equal(pinned, P.U0 * 3)
    s.step(3)
    blob, _, _ = s.get_state()
    U3, t3, _ = s.moments()
    r = gpu.Solver(P, precision="fp64", basis=2)
    r.set_state(blob)
    U, t, steps = r.moments()
    assert t == t3 and steps == 3 and np.array_equal(U, U3)
    s.close()
    r.close()
