"""The kernels' tiles on the CPU, lane by lane (lane_order.cpp): between two
synchronisations the lanes of a wave, and the waves of a block, may run in any
order. The right-hand side, a Runge-Kutta stage with its pushed ghosts and the
constraints are bitwise the same for three orders of lanes and both orders of
waves, and match the oracle by the rule of the parity tests (1e-12 of each
gridfunction's scale beyond twice the FP64 oracle's error). Walks of other bands
give the same."""
import ctypes
import os
import subprocess

import numpy as np
import pytest

from gpu_helpers import check_parity, ld
from oracle import oracle as orc
from paper_2505_00097_amd import capi
from paper_2505_00097_amd import workloads as wl

HERE = os.path.dirname(os.path.abspath(__file__))
ROCM = os.environ.get("ROCM_PATH", "/opt/rocm")
TOL = 1e-12
DISS = (0.99, 0.3)


def _build(variant, out):
    cmd = [os.path.join(ROCM, "lib", "llvm", "bin", "clang++"), "-x", "c++", "-std=c++17", "-O1", "-mavx2", "-mfma",
           "-ffp-contract=on", "-Wno-everything", "-fPIC", "-shared", "-D__HIP_PLATFORM_AMD__",
           f"-I{ROCM}/include", f"-DVARIANT={variant}", os.path.join(HERE, "lane_order.cpp"), "-o", out]
    subprocess.run(cmd, check=True)
    return ctypes.CDLL(out)


# each order of differences, with two phi planes and more, on whole, cut and ragged 16 x 4 patches
@pytest.mark.parametrize("coord,N,ng,bc", [
    (wl.SINH_SPHERICAL, (18, 7, 4), 3, 0), (wl.SINH_CYLINDRICAL, (17, 2, 9), 3, 0),
    (wl.SINH_CYLINDRICAL, (18, 4, 6), 5, 1), (wl.SPHERICAL, (33, 5, 2), 5, 1)])
def test_results_do_not_depend_on_the_order_of_lanes(tmp_path, coord, N, ng, bc):
    two = N[1 if coord == wl.SINH_CYLINDRICAL else 2] == 2
    lib = _build(2 * coord + two + (6 if ng == 5 else 0), str(tmp_path / "tiles.so"))
    ampl, w = (2.0, 2.0, 3.0), (0.3,) * 3
    par = capi.GridParams(coord, (ctypes.c_int * 3)(*N), ng, (ctypes.c_double * 3)(*ampl), (ctypes.c_double * 3)(*w),
                          0.5, bc)
    gp = capi.GaugeParams(2.0, 0, *DISS)
    og = orc.Grid(coord, N, ampl=ampl, sinhw=w, ng=ng, diss=DISS)
    ol = og.twin()
    I = og.interior()
    y = og.apply_bcs(wl.smooth_random_state(og.n, seed=7))
    base = wl.smooth_random_state(og.n, seed=8)
    dp = lambda a: a.ctypes.data_as(ctypes.POINTER(ctypes.c_double))

    def run(what, order, band=4):
        out, aux = np.full(y.shape, np.nan), np.full((9,) + y.shape[1:], np.nan)
        rc = lib.run_tiles(ctypes.byref(par), ctypes.byref(gp), what, order, band, dp(y), dp(base), ctypes.c_double(1e-3),
                           dp(out), dp(aux))
        assert rc == 0, (what, order, rc)
        return np.concatenate([out, aux])

    res = []
    for what in range(3):
        a = [run(what, order) for order in range(3)]
        for order in (1, 2):
            assert np.array_equal(a[0], a[order], equal_nan=True), (what, order)
        for band in (1, 2, 16):
            assert np.array_equal(a[0], run(what, 0, band), equal_nan=True), (what, "band", band)
        res.append(a[0])
    rhs, stage, con = res[0][:24], res[1][:24], res[2][:7]
    sl = (slice(None),) + I
    check_parity(f"lane order rhs {coord} {N} ng {ng}", rhs, og.rhs(y, eta=2.0), ol.rhs(ld(y), eta=2.0), I, TOL,
                 names=orc.GF_NAMES)
    np.testing.assert_allclose(stage[sl], base[sl] + 1e-3 * rhs[sl], rtol=1e-15, atol=1e-15)
    # pushed ghosts, where the kernel pushes: some of the ghosts, as the oracle fills them (integer
    # weights of up to 9 and 961 terms; the other ghosts were not written)
    pushed = ~np.isnan(stage[0])
    pushed[I] = False
    assert pushed.any() == (two or ng == 3)
    if bc == 0:
        full = og.apply_bcs(np.where(np.isnan(stage), 0.0, stage))
        np.testing.assert_allclose(stage[:, pushed], full[:, pushed], rtol=0, atol=961 * 9 * 2.3e-16 * np.abs(base).max())

    def cons(o, v):
        Hc, M, Cc = o.constraints(v)
        return np.concatenate([Hc[None], M, Cc])

    check_parity(f"lane order constraints {coord} {N} ng {ng}", con, cons(og, y), cons(ol, ld(y)), I, TOL,
                 groups=[[0], [1, 2, 3], [4, 5, 6]])
