"""The launch of an ensemble's right-hand-side kernel follows the tiles of the
current job set: blocks_per_cu x CUs striding blocks for up to 8 tiles per
block, one block per tile (rounded up by at most 1/32) beyond, whatever the
batch held before. Results are bitwise those of single steps."""
import pytest

from paper_2505_00097_amd import workloads as wl

pytestmark = pytest.mark.gpu

LONG, SHORT = (256, 128, 32), (37, 11, 6)  # 16 x 32 x 32 and 3 x 3 x 6 tiles
TILES = {LONG: 16384, SHORT: 54}


def _jobs(sizes):
    import torch
    from paper_2505_00097_amd import capi
    grids = [capi.Grid(wl.SINH_SPHERICAL, N, (10.0,) * 3, (0.2,) * 3) for N in sizes]
    ys = [g.state() for g in grids]
    for g, y in zip(grids, ys):
        capi.set_initial_data_brill_lindquist(g.h, [0.6, 0.4], [(0.7, 0.1, 0.0), (-0.7, 0.0, 0.2)], y)
    torch.cuda.synchronize()
    return grids, ys, [g.workspace() for g in grids]


def _cus():
    import torch
    return torch.cuda.get_device_properties(0).multi_processor_count


def _step(b, jobs, active=None):
    import torch
    from paper_2505_00097_amd import capi
    grids, ys, wss = jobs
    capi.batch_step(b, ys, wss, [g.dt for g in grids], active=active, nsteps=1)
    torch.cuda.synchronize()
    return capi.batch_get_info(b)


def test_a_shrunk_list_launches_as_a_fresh_one():
    print("launch blocks: shrunk list", flush=True)
    import torch
    from paper_2505_00097_amd import capi
    jobs = _jobs([LONG, SHORT])
    grids, ys, wss = jobs
    solo = [y.clone() for y in ys]
    b = capi.batch_create([g.h for g in grids])
    n = sum(TILES.values())
    info = _step(b, jobs)
    assert info.n_tiles == n and n <= info.rhs_blocks <= n + n // 32 + 8
    info = _step(b, jobs, active=[False, True])
    assert info.n_tiles == TILES[SHORT]
    fresh = capi.batch_create([grids[1].h])
    spare = (grids[1:], [ys[1].clone()], wss[1:])
    assert info.rhs_blocks == _step(fresh, spare).rhs_blocks == 4 * _cus()
    info = _step(b, jobs)  # the long list again
    assert n <= info.rhs_blocks <= n + n // 32 + 8
    for g, y, ws, s, k in zip(grids, ys, wss, solo, (2, 3)):
        for _ in range(k):
            capi.rk4_step(g.h, s, ws, g.dt)
        assert torch.equal(y, s), g.N
    capi.batch_destroy(fresh)
    capi.batch_destroy(b)


@pytest.mark.parametrize("size,bpc", [(SHORT, 1), (SHORT, 2), (SHORT, 4), (SHORT, 0), (LONG, 1), (LONG, 4), (LONG, 0)])
def test_blocks_per_cu_sets_the_launch(size, bpc):
    print("launch blocks:", size, bpc, flush=True)
    from paper_2505_00097_amd import capi
    jobs = _jobs([size])
    b = capi.batch_create([jobs[0][0].h])
    capi.batch_set_blocks_per_cu(b, bpc)
    blocks, n = _step(b, jobs).rhs_blocks, TILES[size]
    if bpc and n <= 8 * bpc * _cus():
        assert blocks == bpc * _cus()
    else:
        assert n <= blocks <= n + n // 32 + 8
    capi.batch_destroy(b)


def _tuned(grids, ys, wss, cache):
    import torch
    from paper_2505_00097_amd import capi
    b = capi.batch_create([g.h for g in grids], tune_cache_path=cache)
    capi.batch_set_launch_tuning(b, True)
    capi.batch_step(b, ys, wss, [g.dt for g in grids], nsteps=1)
    torch.cuda.synchronize()
    info = capi.batch_get_info(b)
    capi.batch_destroy(b)
    return info


@pytest.mark.parametrize("sizes,launches", [([LONG, SHORT], 3), ([LONG], 6), ([SHORT], 12)])
def test_launch_tuning_times_each_launch_once(tmp_path, sizes, launches):
    """Of the blocks per CU {2, 4, 8, one per tile}, those that come to one
    launch are one candidate (each at three graph lengths); a stored choice is
    taken where it comes to the launch that was timed, and timed again where
    not."""
    print("launch tuning:", sizes, flush=True)
    jobs = _jobs(sizes)
    path = tmp_path / "tiles.json"
    first = _tuned(*jobs, str(path))
    assert first.launch_candidates == launches and not first.launch_from_cache
    again = _tuned(*jobs, str(path))
    assert again.launch_from_cache and again.rhs_blocks == first.rhs_blocks
    stored = f'"blocks": {first.rhs_blocks}}}'
    assert path.read_text().count(stored) == 1
    path.write_text(path.read_text().replace(stored, f'"blocks": {first.rhs_blocks + 8}}}'))
    assert not _tuned(*jobs, str(path)).launch_from_cache
