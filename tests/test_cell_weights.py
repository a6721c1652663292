"""Branches of the per-cell split, against the oracle on the host (no GPU):
the weights' polynomial (arguments up to 1.02) and the exponential form beyond
it, and MHD's coupling to the cleaning pair with c_h far from the wave speeds
(one common denominator), close to them and on one of them (divided
differences). Tolerances are those the split is held to elsewhere: 2e-12 of the
flux in FP64, 1e-8 where speeds coincide, and in FP32 1e-6 times the
conditioning of a difference quotient at that distance."""
import numpy as np
import pytest

from test_cell_math import cc, cc_split, cfg, prm, rand_state  # noqa: F401


@pytest.mark.parametrize("system,dim", [("sw", 2), ("euler", 1), ("euler", 2), ("mhd", 2), ("linear", 1)])
@pytest.mark.parametrize("zmax", [1e-3, 0.5, 1.0, 1.0199, 1.0201, 1.5, 4.0])
def test_weights_on_both_sides_of_the_polynomials_range(oracle, cc, system, dim, zmax):  # noqa: F811
    O = oracle
    rng = np.random.default_rng(31)
    gamma = 2.0 if system == "mhd" else 1.4
    for k in (2.0, 8.0):
        if system == "linear":
            cf = O.make_config(system="linear", dim=1, n=(8, 1), adv=(0.7, 0.0), k=k)
            pr = prm(gamma=gamma, k=k)
            pr[3] = 0.7
        else:
            cf = cfg(O, system, dim, k=k)
            pr = prm(gamma=gamma, k=k)
        for _ in range(10):
            U = rand_state(system, dim, rng) if system != "linear" else np.array([rng.uniform(0.5, 2.0)])
            ch = 0.0
            if system == "mhd":
                ch = 6.0 * max(O.fast_speed(cf, d, U) for d in range(dim))
            for d in range(dim):
                lam7 = np.abs(O.eigenvalues(cf, d, U, ch))
                top = np.sort(lam7)[-3] if system == "mhd" else lam7.max()  # the fastest wave besides the pair
                Lam = 0.5 * k * top / zmax
                Fpo, Fmo = O.split(cf, d, U, ch, lam=Lam)
                for size, tol in ((8, 2e-12), (4, 3e-6)):
                    F, D = cc_split(cc, size, system, dim, d, U, pr, Lam, ch)
                    sc = np.max(np.abs(F)) + 1.0
                    assert np.max(np.abs((0.5 * F + D) - Fpo)) < tol * sc, (k, size)
                    assert np.max(np.abs((0.5 * F - D) - Fmo)) < tol * sc, (k, size)


@pytest.mark.parametrize("ratio", [0.4, 0.9, 1.1, 1.6, 1.99, 2.01, 3.0, 6.0])
@pytest.mark.parametrize("dim", [1, 2])
def test_mhd_cleaning_speed_near_and_far_from_the_waves(oracle, cc, dim, ratio):  # noqa: F811
    """ratio: c_h over the fastest wave."""
    O = oracle
    rng = np.random.default_rng(32)
    cf = cfg(O, "mhd", dim)
    pr = prm(gamma=2.0)
    for _ in range(20):
        U = rand_state("mhd", dim, rng)
        for d in range(dim):
            u = U[1 + d] / U[0]
            top = abs(u) + O.fast_speed(cf, d, U)
            ch = top * ratio
            Lam = 1.1 * max(top, ch)
            Fpo, _ = O.split(cf, d, U, ch, lam=Lam)
            F, D = cc_split(cc, 8, "mhd", dim, d, U, pr, Lam, ch)
            sc = np.max(np.abs(F)) + 1.0
            # distance of the nearest wave from +-c_h, relative
            ev = O.eigenvalues(cf, d, U, ch)
            gap = np.sort(np.abs(np.abs(ev) - ch) / ch)[2]
            assert np.max(np.abs((0.5 * F + D) - Fpo)) < (2e-12 / gap if gap > 1e-4 else 1e-8) * sc
            F, D = cc_split(cc, 4, "mhd", dim, d, U, pr, Lam, ch)
            assert np.max(np.abs((0.5 * F + D) - Fpo)) < 1e-6 / max(gap, 1e-3) * sc


@pytest.mark.parametrize("dim", [1, 2])
def test_mhd_cleaning_speed_on_the_fast_wave(cc, oracle, dim):  # noqa: F811
    """With c_h on a wave the Jacobian has no full set of eigenvectors, so the
    oracle's route does not apply; the split is a smooth function of c_h and
    equals the mean of its neighbours' to second order."""
    O = oracle
    rng = np.random.default_rng(33)
    cf = cfg(O, "mhd", dim)
    pr = prm(gamma=2.0)
    for _ in range(20):
        U = rand_state("mhd", dim, rng)
        for d in range(dim):
            ch = abs(U[1 + d] / U[0]) + O.fast_speed(cf, d, U)
            Lam = 1.1 * ch
            D = [cc_split(cc, 8, "mhd", dim, d, U, pr, Lam, ch * (1 + e))[1] for e in (-1e-5, 0.0, 1e-5)]
            assert np.max(np.abs(0.5 * (D[0] + D[2]) - D[1])) < 1e-8 * (np.max(np.abs(D[1])) + 1.0)
