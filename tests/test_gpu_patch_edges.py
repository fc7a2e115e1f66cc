"""The right-hand side and the constraints where a 16 x 4 patch of the kernels
is cut: grids one point short of, at and past a patch along both directions,
and thinner than one, with two and more phi planes, at both orders. Reference
and tolerance are those of the parity tests (the extended-precision oracle,
1e-12 of each gridfunction's scale beyond twice the FP64 oracle's error)."""
import numpy as np
import pytest

from gpu_helpers import check_parity, ld, to_cpu, to_gpu
from oracle import oracle as orc
from paper_2505_00097_amd import workloads as wl

pytestmark = pytest.mark.gpu
TOL = 1e-12
DISS = (0.99, 0.3)

# (points along i0, along the other direction e, phi planes)
SIZES = [(15, 5, 3), (16, 4, 4), (17, 3, 5), (33, 9, 2), (3, 13, 6), (18, 7, 2)]


@pytest.mark.parametrize("coord", [wl.SINH_SPHERICAL, wl.SINH_CYLINDRICAL, wl.SPHERICAL])
@pytest.mark.parametrize("ng", [3, 5])
@pytest.mark.parametrize("n0,ne,nphi", SIZES)
def test_patch_edges(coord, ng, n0, ne, nphi):
    nphi += nphi % 2  # the inner maps need an even number of planes
    n0, ne = max(n0, ng), max(ne, ng)
    N = (n0, nphi, ne) if coord == wl.SINH_CYLINDRICAL else (n0, ne, nphi)
    print("patch edges", coord, N, ng, flush=True)
    import torch
    from paper_2505_00097_amd import capi
    ampl = (2.0, 2.0, 3.0)
    g = capi.Grid(coord, N, ampl, (0.3,) * 3, nghosts=ng)
    og = orc.Grid(coord, N, ampl=ampl, sinhw=(0.3,) * 3, ng=ng, diss=DISS)
    ol = og.twin()
    I = og.interior()
    y = og.apply_bcs(wl.smooth_random_state(og.n, seed=7))
    r = g.state()
    r.zero_()
    capi.bssn_rhs(g.h, to_gpu(y), r, eta=2.0, diss=DISS)
    check_parity(f"patch edges rhs+ko {coord} {N} ng {ng}", to_cpu(r), og.rhs(y, eta=2.0), ol.rhs(ld(y), eta=2.0), I,
                 TOL, names=orc.GF_NAMES)
    out = [g._empty(1), g._empty(3), g._empty(3)]
    for t in out:
        t.zero_()
    capi.constraints(g.h, to_gpu(y), *out)
    torch.cuda.synchronize()

    def cons(o, v):
        H, M, C = o.constraints(v)
        return np.concatenate([H[None], M, C])

    check_parity(f"patch edges constraints {coord} {N} ng {ng}", np.concatenate([to_cpu(t) for t in out]),
                 cons(og, y), cons(ol, ld(y)), I, TOL, groups=[[0], [1, 2, 3], [4, 5, 6]])
