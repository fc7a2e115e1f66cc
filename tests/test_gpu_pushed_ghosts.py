"""Stage ghosts written by the right-hand-side kernel itself (a single grid)
against the ghost kernel (an ensemble): both form the same sums in the same
order, so whole evolutions, every ghost included, are bitwise equal.
The sizes put the sources of outer ghosts inside one 16 x 4 patch, across two
(N0 or N_e one or two points past a multiple: those ghosts stay with the ghost
kernel) and in grids smaller than a patch; both boundaries, both orders, all
coordinate families, with and without the stages that mix two states."""
import pytest

from paper_2505_00097_amd import workloads as wl

pytestmark = pytest.mark.gpu

CASES = [
    (wl.SINH_CYLINDRICAL, (16, 2, 8), 3), (wl.SINH_CYLINDRICAL, (17, 2, 21), 3), (wl.SINH_CYLINDRICAL, (18, 6, 22), 3),
    (wl.SINH_CYLINDRICAL, (35, 2, 11), 5), (wl.SINH_CYLINDRICAL, (5, 4, 6), 5), (wl.SINH_CYLINDRICAL, (3, 2, 3), 3),
    (wl.SINH_SPHERICAL, (33, 9, 2), 3), (wl.SINH_SPHERICAL, (20, 7, 6), 3), (wl.SINH_SPHERICAL, (49, 6, 2), 5),
    (wl.SPHERICAL, (34, 4, 4), 3), (wl.SPHERICAL, (31, 13, 2), 3), (wl.SPHERICAL, (7, 5, 2), 5),
]


@pytest.mark.parametrize("bc", [0, 1])
@pytest.mark.parametrize("coord,N,ng", CASES)
def test_pushed_ghosts_equal_the_ghost_kernel(coord, N, ng, bc):
    print("pushed ghosts", coord, N, ng, bc, flush=True)
    import torch
    from paper_2505_00097_amd import capi
    g = capi.Grid(coord, N, (10.0,) * 3, (0.3,) * 3, bc_kind=bc, nghosts=ng)
    y0 = torch.from_numpy(wl.smooth_random_state(g.n, seed=31)).cuda()
    capi.apply_bcs(g.h, y0)
    ws = g.workspace()
    for integrator, diss in ((capi.RK4, (0.0, 0.0)), (capi.SSPRK3, (0.99, 0.3))):
        y, yb = y0.clone(), y0.clone()
        ws.fill_(float("nan"))  # every ghost that a stage reads is written within the step
        capi.evolve(g.h, y, ws, 0.1 * g.dt, 2, integrator=integrator, diss=diss)
        torch.cuda.synchronize()
        ws.fill_(float("nan"))
        b = capi.batch_create([g.h], diss=diss)
        capi.batch_set_integrator(b, integrator)
        capi.batch_step(b, [yb], [ws], [0.1 * g.dt], nsteps=2)
        torch.cuda.synchronize()
        capi.batch_destroy(b)
        assert torch.isfinite(y).all()
        assert torch.equal(y, yb), integrator
