"""Launch shapes of solves that keep U (omega = 1): every shape a caller can ask
for gives the same bits."""
import numpy as np
import pytest

from test_gpu_omega1 import populations, run, state1d, state2d

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("system,prec", [("sw", "fp32"), ("euler", "fp32"), ("euler", "fp64")])
@pytest.mark.parametrize("bc", ["periodic", "zero_gradient", "characteristic"])
def test_one_workgroup_lanes_are_bitwise_the_launch_path(gpu, system, prec, bc):
    """256 lanes of up to 4 cells, 512 of up to 2 and 1024, with partly filled
    wavefronts and wavefronts past the end of the grid."""
    for n in (2, 255, 257, 300, 511, 513, 640, 767, 769, 1000, 1024):
        P = state1d(system, n, n, bc=(bc, bc))
        print(f"[case] {system} {n} {prec} {bc}", flush=True)
        ref = run(gpu, P, prec, 23, small_grid=-1)
        for lanes in (256, 512, 1024):
            got = run(gpu, P, prec, 23, small_grid=lanes)
            assert got[1:3] == ref[1:3] and np.array_equal(got[0], ref[0]), (n, lanes)
            assert np.array_equal(populations(got[3], P), populations(ref[3], P)), (n, lanes)


@pytest.mark.parametrize("system,prec", [("sw", "fp32"), ("euler", "fp32"), ("mhd", "fp32"), ("mhd", "fp64")])
def test_rows_and_strips_give_identical_results(gpu, system, prec):
    """1 to 45 rows a wavefront (more than one batch of halo rows, a last band
    that is not full), asked for as rows of 64, 128 or 256 columns."""
    P = state2d(system, 200, 90, 5, bc=("zero_gradient", "periodic"))
    ref = run(gpu, P, prec, 12)
    for width, rows in ((64, 4), (64, 12), (64, 180), (128, 5), (128, 66), (256, 7), (256, 33), (0, 45)):
        got = run(gpu, P, prec, 12, strip_width=width, band_rows=rows)
        assert got[1:3] == ref[1:3] and np.array_equal(got[0], ref[0]), (width, rows)
        assert np.array_equal(populations(got[3], P), populations(ref[3], P)), (width, rows)


@pytest.mark.parametrize("prec,basis", [("fp64", 0), ("fp32", 2), ("fp32", 3)])
def test_checkpoints_follow_the_state(gpu, prec, basis):
    """The populations of a checkpoint are the current state's, whatever was
    rebuilt, initialized or restored before: asked for twice, at the same step
    count of another initial state, and before the first step after others."""
    A, B = (state2d("euler", 70, 20, seed, bc=("periodic", "periodic")) for seed in (1, 2))
    ref = {(k, n): populations(run(gpu, P, prec, n, basis=basis)[3], P) for k, P in (("a", A), ("b", B)) for n in (0, 4, 7)}
    s = gpu.Solver(A, precision=prec, basis=basis)
    dt = np.float32 if prec == "fp32" else np.float64

    def check(key):
        for _ in range(2):
            blob = s.get_state()[0]
            assert np.array_equal(populations(blob[:-128].view(dt), A), ref[key]), key
        return blob

    s.init(A.U0)
    check(("a", 0))
    s.step(4)
    a4 = check(("a", 4))
    s.step(3)
    check(("a", 7))
    s.init(B.U0)
    s.step(4)
    check(("b", 4))
    s.init(A.U0)
    check(("a", 0))
    s.init(B.U0)
    s.step(7)
    s.set_state(a4)
    check(("a", 4))
    s.step(3)
    check(("a", 7))
    s.init(B.U0)
    check(("b", 0))
    s.close()
