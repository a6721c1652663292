"""Launch shapes the library chooses by itself, on the host (no GPU), through the
host check library, which compiles the functions the library uses."""
import ctypes

import pytest

from test_cell_math import KIND
from test_row_layout import CC


@pytest.fixture(scope="module")
def cc():
    import os
    if not os.path.exists(CC):
        from paper_2608_04283_amd import build
        build.build_cellcheck()
    L = ctypes.CDLL(CC)
    ll = ctypes.c_longlong
    L.vklb_cc_default_uband.argtypes = [ctypes.c_int, ctypes.c_int, ll, ll]
    L.vklb_cc_ustep_waves.argtypes = [ll, ll, ctypes.c_int]
    L.vklb_cc_ustep_waves.restype = ll
    L.vklb_cc_uside.argtypes = [ctypes.c_int, ctypes.c_int, ll]
    L.vklb_cc_tune_candidates.argtypes = [ctypes.c_int] * 3 + [ll, ll, ctypes.c_double, ctypes.c_int, ctypes.c_void_p,
                                                               ctypes.c_int]
    L.vklb_cc_uband_of.argtypes = [ctypes.c_int, ctypes.c_int]
    L.vklb_cc_default_shape.argtypes = [ctypes.c_int, ctypes.c_int, ll, ll, ctypes.c_int, ctypes.c_void_p]
    L.vklb_cc_default_shape.restype = None
    L.vklb_cc_keeps_u.argtypes = [ctypes.c_int] * 3 + [ctypes.c_double]
    L.vklb_cc_uwg_lanes.argtypes = [ctypes.c_int, ll, ctypes.c_int]
    return L


SIDES = [1, 2, 3, 63, 64, 65, 128, 200, 258, 300, 333, 500, 580, 724, 819, 1000, 1024, 1199, 1289, 1532, 2048, 4096]


@pytest.mark.parametrize("system", ["sw", "euler", "mhd", "linear"])
@pytest.mark.parametrize("prec", [4, 8])
def test_default_rows_of_u_solves_are_one_round_of_wavefronts(cc, system, prec):
    """The fewest rows whose wavefronts are all resident at once, whatever the
    sides are: at most 16 (MHD 32), one row where a row each is at most 1024."""
    resident = 1024 * {("mhd", 4): 2, ("mhd", 8): 1}.get((system, prec), 4 if prec == 4 else 2)
    most = 32 if system == "mhd" else 16
    for nx in SIDES:
        for ny in SIDES:
            rows = cc.vklb_cc_default_uband(KIND[system], prec, nx, ny)
            waves = [cc.vklb_cc_ustep_waves(nx, ny, r) for r in range(1, most + 1)]
            if waves[0] <= 1024:
                want = 1
            else:
                want = next((r for r in range(2, most + 1) if waves[r - 1] <= resident), most)
            assert rows == want, (nx, ny)


@pytest.mark.parametrize("system", ["sw", "euler", "linear"])
def test_one_workgroup_lanes_are_the_ones_asked_for(cc, system):
    """Every grid of up to 1024 cells runs with 256, 512 or 1024 lanes as asked
    (4, 2 or 1 cells each); without a request with the fastest measured, and
    larger ones with 1024 of two cells."""
    for n in list(range(1, 1025, 13)) + [256, 257, 512, 513, 1024]:
        for lanes in (256, 512, 1024):
            assert cc.vklb_cc_uwg_lanes(KIND[system], n, lanes) == lanes, n
        assert cc.vklb_cc_uwg_lanes(KIND[system], n, 0) == (256 if n <= 256 else 512)
    for n in (1025, 2048):
        assert [cc.vklb_cc_uwg_lanes(KIND[system], n, k) for k in (0, 256, 512, 1024)] == [1024] * 4


def test_one_workgroup_lanes_of_mhd_hold_one_cell_each(cc):
    for n in (1, 256, 257, 512, 513, 768):
        for lanes in (0, 256, 512, 1024):
            got = cc.vklb_cc_uwg_lanes(KIND["mhd"], n, lanes)
            assert got >= n and got == (lanes if lanes >= n else 256 if n <= 256 else 512 if n <= 512 else 1024)


@pytest.mark.parametrize("system,prec,most", [("sw", 4, 4), ("euler", 4, 4), ("euler", 8, 4), ("linear", 8, 4), ("mhd", 4, 2),
                                              ("mhd", 8, 1)])
def test_tiles_of_256_only_where_they_save_a_workgroup_a_unit(cc, system, prec, most):
    """Just below k x 65,536 cells, for the k at which it measured faster, and
    never above."""
    ends = [f * k + d for k in range(1, 260) for f in (254 * 256, 65536) for d in (0, 1)]
    for n in ends + list(range(1, 1 << 25, 9973)):
        want = any(254 * 256 * k < n <= 65536 * k for k in range(1, most + 1))
        assert bool(cc.vklb_cc_uside(KIND[system], prec, n)) == want, n


def candidates(cc, system, prec, nx, ny=0, omega=1.0, pool=False):
    out = (ctypes.c_int * 800)()
    n = cc.vklb_cc_tune_candidates(KIND[system], prec, 2 if ny else 1, nx, max(ny, 1), omega, int(pool), out, 200)
    assert 0 < n <= 200
    c = [tuple(out[4 * i:4 * i + 4]) for i in range(n)]
    assert len(set(c)) == n
    return c


@pytest.mark.parametrize("pool", [False, True])
@pytest.mark.parametrize("omega", [1.0, 1.5])
@pytest.mark.parametrize("prec", [4, 8])
@pytest.mark.parametrize("system", ["sw", "euler", "mhd", "linear"])
def test_the_tuner_times_the_default_2d_shape(cc, system, prec, omega, pool):
    for nx in SIDES + [129, 257, 8192]:
        for ny in SIDES:
            c = candidates(cc, system, prec, nx, ny, omega, pool)
            if omega == 1.0:
                rows = [cc.vklb_cc_uband_of(b, w) for w, b, _, _ in c]
                rule = cc.vklb_cc_default_uband(KIND[system], prec, nx, ny)
                assert len(set(rows)) == len(rows) and (rule in rows or pool and rule < 4)
                assert not pool or min(rows) == 4  # (a full pool runs taller bands faster)
            else:
                d = (ctypes.c_int * 3)()
                cc.vklb_cc_default_shape(KIND[system], prec, nx, ny, 128 if pool else 0, d)
                assert tuple(d) + (0,) in c, (nx, ny)


def test_rows_of_a_wavefront_of_a_u_solve(cc):
    """A workgroup's four wavefronts share band_rows rows of strip_width columns."""
    for band, width, rows in ((1, 0, 1), (40, 0, 40), (40, 256, 40), (40, 77, 40), (40, 128, 20), (5, 128, 3),
                              (4, 64, 1), (5, 64, 2), (64, 64, 16), (3, 64, 1), (2**31 - 1, 64, 4096), (5000, 0, 4096)):
        assert cc.vklb_cc_uband_of(band, width) == rows


@pytest.mark.parametrize("omega", [1.0, 1.5])
def test_the_tuner_times_each_1d_shape_once(cc, omega):
    for n in (1, 200, 256, 257, 513, 1024):
        lanes = [c[3] for c in candidates(cc, "euler", 4, n, omega=omega)]
        assert lanes == [256, 512, 1024]
        assert [cc.vklb_cc_uwg_lanes(KIND["euler"], n, k) for k in lanes] == lanes
        assert cc.vklb_cc_uwg_lanes(KIND["euler"], n, 0) in lanes
    assert [c[0] for c in candidates(cc, "euler", 4, 3000, omega=omega)] == ([256] if omega == 1.0 else [256, 512])


def test_the_rule_of_the_solves_that_keep_u_is_the_same_in_python(cc):
    """serving.keeps_u (the algorithmic bytes of the benchmark and of the served
    stream) states the library's rule."""
    from paper_2608_04283_amd import inputs as I
    from paper_2608_04283_amd.serving import alg_bytes, keeps_u
    for system in KIND:
        for dim in (1, 2):
            for prec, size in (("fp32", 4), ("fp64", 8)):
                for omega in (1.0, 1.0 + 2.0 ** -52, 0.9, 1.5, 2.0):
                    P = I.Problem(name="p", system=system, dim=dim, n=(8,) * dim, omega=omega)
                    u = bool(cc.vklb_cc_keeps_u(KIND[system], size, dim, omega))
                    assert keeps_u(P, prec) == u
                    assert alg_bytes(P, prec) == 2 * P.p * size * (1 if u else P.Q)
