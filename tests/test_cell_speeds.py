"""FP64 wave speeds of the per-cell arithmetic (vklb_cell.hpp, on the host): a
quotient is rounded as a division rounds it, so they are bit for bit what
numpy's float64 gives for the same expressions. (The host build does not fuse
products into sums.)"""
import ctypes

import numpy as np
import pytest

from test_cell_math import KIND, _p, cc, prm, rand_state  # noqa: F401


def speeds(system, dim, U, gamma):
    f = np.float64
    m2 = f(0.0)
    for k in range(dim if system == "euler" else 3):
        m2 = m2 + U[1 + k] * U[1 + k]
    if system == "euler":
        p = (gamma - f(1)) * (U[dim + 1] - f(0.5) * (m2 / U[0]))
        c = np.sqrt(gamma * p / U[0])
        return max(abs(U[1 + d] / U[0]) + c for d in range(dim)), f(0.0)
    B = U[5:8]
    B2 = B[0] * B[0] + B[1] * B[1] + B[2] * B[2]
    p = (gamma - f(1)) * (U[4] - f(0.5) * (m2 / U[0]) - f(0.5) * B2)
    lam = cf = f(0.0)
    for d in range(dim):
        a2 = gamma * p / U[0]
        bn2 = B[d] * B[d] / U[0]
        s, t = B[(d + 1) % 3], B[(d + 2) % 3]
        bt2 = (s * s + t * t) / U[0]
        disc = np.sqrt((a2 - bn2) * (a2 - bn2) + bt2 * (f(2) * a2 + f(2) * bn2 + bt2))
        fast = np.sqrt(f(0.5) * (a2 + bn2 + bt2 + disc))
        lam, cf = max(lam, abs(U[1 + d] / U[0]) + fast), max(cf, fast)
    return lam, cf


@pytest.mark.parametrize("system,dim", [("euler", 1), ("euler", 2), ("mhd", 1), ("mhd", 2)])
def test_fp64_speeds_round_each_quotient_once(cc, system, dim):  # noqa: F811
    rng = np.random.default_rng(71)
    gamma = np.float64(2.0 if system == "mhd" else 1.4)
    for scale in (1.0, 1e-5, 1e4):
        for _ in range(500):
            U = np.asarray(rand_state(system, dim, rng), dtype=np.float64) * scale
            U[5:8] /= np.sqrt(scale)  # (MHD: the field's pressure scales as the others)
            lam, cfm = ctypes.c_double(), ctypes.c_double()
            cc.vklb_cc_speeds(8, KIND[system], dim, _p(U), _p(prm(gamma=gamma)), ctypes.byref(lam), ctypes.byref(cfm))
            ref = speeds(system, dim, U, gamma)
            assert np.isfinite(ref).all() and (lam.value, cfm.value) == ref
