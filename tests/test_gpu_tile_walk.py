"""The walk of the 16 x 4 tiles: bands of 1, 4 and 16 rows and one wider than
the grid, on grids of several full and ragged bands with cut patches (the
per-lane form of the stage combination) and whole ones (row pairs). The
right-hand side with its aux arrays and whole steps are bitwise the same, for
a single grid and in an ensemble whose bands come from the cache file."""
import json

import pytest

from paper_2505_00097_amd import workloads as wl

pytestmark = pytest.mark.gpu

DISS = (0.99, 0.3)
BANDS = (1, 4, 16, 1000)
# tile rows per band run along i1: theta patches of 4 points, or phi planes on cylindrical grids
GRIDS = [(wl.SINH_SPHERICAL, (32, 73, 4), 3), (wl.SPHERICAL, (18, 90, 2), 3), (wl.SINH_CYLINDRICAL, (35, 22, 9), 3),
         (wl.SINH_CYLINDRICAL, (16, 18, 8), 5), (wl.SPHERICAL, (33, 41, 6), 5)]


def _grid(coord, N, ng):
    import torch
    from paper_2505_00097_amd import capi
    g = capi.Grid(coord, N, (10.0,) * 3, (0.3,) * 3, nghosts=ng)
    y = torch.from_numpy(wl.smooth_random_state(g.n, seed=17)).cuda()
    capi.apply_bcs(g.h, y)
    return g, y


@pytest.mark.parametrize("coord,N,ng", GRIDS)
def test_bands_do_not_change_a_grid(coord, N, ng):
    print("tile walk", coord, N, ng, flush=True)
    import torch
    from paper_2505_00097_amd import capi
    g, y0 = _grid(coord, N, ng)
    ws, ref = g.workspace(), None
    for band in BANDS:
        capi.grid_set_tile(g.h, 6, 0, band)
        out = [g.state().fill_(-7.0), g.aux().fill_(-7.0), y0.clone(), y0.clone()]
        capi.bssn_rhs(g.h, y0, out[0], out[1], diss=DISS)
        capi.rk4_step(g.h, out[2], ws, 0.1 * g.dt)
        capi.ssprk3_step(g.h, out[3], ws, 0.1 * g.dt, diss=DISS)
        torch.cuda.synchronize()
        if ref is None:
            ref = out
            assert all(torch.isfinite(t).all() for t in ref)
            I = (slice(None),) + tuple(slice(ng, ng + N[d]) for d in (2, 1, 0))
            r = ref[0].view((24,) + tuple(g.n[d] for d in (2, 1, 0)))
            assert not (r[I] == -7.0).any()  # every interior point is written
        for a, b in zip(ref, out):
            assert torch.equal(a, b), band


@pytest.mark.parametrize("band", BANDS)
def test_bands_do_not_change_an_ensemble(tmp_path, band):
    print("tile walk, ensemble", band, flush=True)
    import torch
    from paper_2505_00097_amd import capi
    jobs = [_grid(*p) for p in GRIDS]
    arch = torch.cuda.get_device_properties(0).gcnArchName.split(":")[0]
    path = tmp_path / "tiles.json"
    path.write_text('{"bhah_tile_cache": 1, "entries": [\n' + ",\n".join(
        json.dumps({"arch": arch, "coord": c, "N": list(N), "lx": 6, "ly": 0, "band": band, "us": 1.0})
        for c, N, _ in GRIDS) + "\n]}\n")
    ys, wss = [y.clone() for _, y in jobs], [g.workspace() for g, _ in jobs]
    b = capi.batch_create([g.h for g, _ in jobs], diss=DISS, tune_cache_path=str(path))
    capi.batch_step(b, ys, wss, [0.1 * g.dt for g, _ in jobs], nsteps=1)
    torch.cuda.synchronize()
    assert [capi.batch_get_tile(b, j)[2] for j in range(len(jobs))] == [band] * len(jobs)
    capi.batch_destroy(b)
    for (g, y), yb, ws in zip(jobs, ys, wss):
        capi.rk4_step(g.h, y, ws, 0.1 * g.dt, diss=DISS)
        torch.cuda.synchronize()
        assert torch.equal(y, yb), g.N
