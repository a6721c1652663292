"""Solves with omega = 1 keep U alone (vklb_omega1.hpp); the populations are
rebuilt for a checkpoint. The general path, which stores them, is one step of
the FP64 grid away: omega = 1 + 2^-52 moves a population by 2^-52 of its
distance from equilibrium, below a rounding. So both paths must agree, in U
and in every population of a checkpoint, up to their roundings: each step
rounds a value a few times, steps x 32 roundings of the largest value of its
field (FP64 2^-53, FP32 2^-24) bound what n steps can differ by."""
import numpy as np
import pytest

from paper_2608_04283_amd import inputs as I

pytestmark = pytest.mark.gpu

TRAILER = 128


def state2d(system, nx, ny, seed, **kw):
    rng = np.random.default_rng(seed)
    X, Y = I.grid2(nx, ny, (0.0, 0.0), (1.0, ny / nx))
    w = lambda: rng.uniform(0.05, 0.2) * np.sin(2 * np.pi * (X + Y * nx / ny + rng.uniform()))
    one = np.ones_like(X)
    gamma = 2.0 if system == "mhd" else 1.4
    if system == "sw":
        U0 = I.sw_state(1.0 + w(), w(), w())
    elif system == "euler":
        U0 = I.euler_state(1.0 + w(), w(), 1.0 + w(), gamma, v=w())
    else:
        U0 = I.mhd_state(1.0 + w(), w(), w(), w(), 1.0 + w(), 0.75 * one + w(), w(), w(), gamma, 0.01 * one)
    return I.Problem(name="omega1", system=system, dim=2, n=(nx, ny), hi=(1.0, ny / nx), gamma=gamma, nu=0.4, U0=U0,
                     **kw)


def state1d(system, n, seed, **kw):
    P = state2d(system, n, 1, seed)
    U0 = P.U0 if system == "mhd" else np.delete(P.U0, 2, axis=0)  # no v in 1D
    return P.with_(dim=1, n=(n,), hi=(1.0, 1.0), nu=0.8, U0=U0, **kw)


def run(gpu, P, prec, steps, **opts):
    s = gpu.Solver(P, precision=prec, **opts)
    s.init()
    s.step(steps)
    U, t, n = s.moments()
    blob, _, _ = s.get_state()
    s.close()
    return U, t, n, blob[:-TRAILER].view(np.float32 if prec == "fp32" else np.float64)


def populations(blob, P):
    """(slots * p, cells) of a checkpoint's blocks of 256 cells; the padding left out."""
    nx, ny = P.n if P.dim == 2 else (P.n[0], 1)
    sx = (nx + 63) // 64 * 64 if P.dim == 2 else nx
    blocks = (sx * ny + 255) // 256
    f = blob.reshape(blocks, -1, 256).transpose(1, 0, 2).reshape(-1, blocks * 256)[:, :sx * ny]
    return f.reshape(-1, ny, sx)[:, :, :nx].reshape(-1, nx * ny)


def agree(P, prec, steps, a, b):
    eps = 2.0 ** -24 if prec == "fp32" else 2.0 ** -53
    tol = 32 * max(1, steps) * eps
    assert a[2] == b[2] == steps and abs(a[1] - b[1]) <= tol * max(b[1], 1e-300)
    top = np.abs(populations(b[3], P)).max()
    assert np.abs(a[0] - b[0]).max() <= tol * np.abs(b[0]).max()
    assert np.abs(populations(a[3], P) - populations(b[3], P)).max() <= tol * top


SHAPES = [(1, 1), (1, 3), (63, 5), (64, 33), (65, 2), (128, 7), (200, 70), (321, 4)]


@pytest.mark.parametrize("bc", ["periodic", "zero_gradient"])
@pytest.mark.parametrize("prec", ["fp32", "fp64"])
@pytest.mark.parametrize("system", ["sw", "euler", "mhd"])
def test_2d_agrees_with_the_path_that_stores_populations(gpu, system, prec, bc):
    for k, (nx, ny) in enumerate(SHAPES):
        for steps, opts in ((0, {}), (1, {}), (14, {"band_rows": 3}), (15, {"band_rows": 40, "basis": 2}),
                            (5, {"basis": 3 if prec == "fp32" else 1})):
            P = state2d(system, nx, ny, 10 + k, bc=(bc, bc), alpha_norm="local" if k % 3 == 2 else "global")
            print(f"[case] {system} {nx}x{ny} {prec} {bc} steps={steps} {opts}", flush=True)
            a = run(gpu, P, prec, steps, **opts)
            b = run(gpu, P.with_(omega=1.0 + 2.0 ** -52), prec, steps, **opts)
            agree(P, prec, steps, a, b)


# one workgroup (1 and 2 cells a lane, partly filled wavefronts), tiles of 254
# cells and their edges, more partials than a wavefront reads, tiles of 256
SIZES = [1, 2, 3, 64, 65, 254, 256, 257, 511, 1000, 2048, 2049, 3000, 65100, 65536, 70000]


@pytest.mark.parametrize("bc", ["periodic", "zero_gradient", "characteristic"])
@pytest.mark.parametrize("prec", ["fp32", "fp64"])
@pytest.mark.parametrize("system", ["sw", "euler", "mhd"])
def test_1d_agrees_with_the_path_that_stores_populations(gpu, system, prec, bc):
    for k, n in enumerate(SIZES):
        if bc == "characteristic" and n < 2:
            continue
        for steps, opts in ((0, {}), (1, {}), (14, {}), (15, {"small_grid": -1}), (6, {"basis": 2}),
                            (5, {"basis": 1, "small_grid": 1024})):
            P = state1d(system, n, 40 + k, bc=(bc, bc), alpha_norm="local" if k % 3 == 2 else "global")
            print(f"[case] {system} {n} {prec} {bc} steps={steps} {opts}", flush=True)
            a = run(gpu, P, prec, steps, **opts)
            b = run(gpu, P.with_(omega=1.0 + 2.0 ** -52), prec, steps, **opts)
            agree(P, prec, steps, a, b)


@pytest.mark.parametrize("system,prec", [("euler", "fp32"), ("euler", "fp64"), ("mhd", "fp32"), ("sw", "fp32")])
@pytest.mark.parametrize("bc", ["periodic", "characteristic"])
def test_1d_checkpoints_between_the_one_workgroup_kernel_and_launches(gpu, system, prec, bc):
    for n in (2, 200, 700, 1500):
        P = state1d(system, n, 7, bc=(bc, bc))
        ref = run(gpu, P, prec, 21)
        for first, second in ((0, -1), (-1, 0), (512, 1024)):
            a = gpu.Solver(P, precision=prec, small_grid=first)
            a.init()
            a.step(10)
            blob, _, _ = a.get_state()
            a.close()
            b = gpu.Solver(P, precision=prec, small_grid=second)
            b.set_state(blob)
            assert np.array_equal(b.get_state()[0], blob)
            b.step(11)
            U, t, steps = b.moments()
            b.close()
            assert steps == 21 and t == ref[1] and np.array_equal(U, ref[0]), (n, first, second)


@pytest.mark.parametrize("basis", [1, 2, 3])
def test_checkpoint_before_and_between_steps(gpu, basis):
    """A checkpoint taken before the first step, straight after a restore, and
    after steps: the restored solve hands the same bytes back and continues
    bit for bit."""
    P = state2d("mhd", 130, 37, 4, bc=("periodic", "zero_gradient"))
    s = gpu.Solver(P, precision="fp32", basis=basis)
    s.init()
    for steps in (0, 3, 4):
        s.step(steps)
        blob, _, _ = s.get_state()
        r = gpu.Solver(P, precision="fp32", basis=basis, band_rows=5)
        r.set_state(blob)
        again, _, _ = r.get_state()
        assert np.array_equal(blob, again)
        r.step(6)
        q = gpu.Solver(P, precision="fp32", basis=basis)
        q.init()
        q.step(s.progress()[1] + 6)
        assert np.array_equal(r.moments()[0], q.moments()[0])
        r.close()
        q.close()
    s.close()
