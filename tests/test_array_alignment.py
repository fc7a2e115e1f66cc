"""Arrays of the C ABI are aligned to 8 bytes. The kernels may take two doubles
of them in one access, but may not claim more than that alignment for it: in
the optimised device IR (compiled here, no GPU needed) every vector access to
global doubles is marked align 8."""
import os
import re
import subprocess

import pytest

from paper_2505_00097_amd import build


@pytest.mark.parametrize("source,part", [("rhs_fused.hip", 0), ("rhs_fused.hip", 7), ("hamiltonian.hip", 1)])
def test_vector_accesses_claim_eight_bytes(tmp_path, source, part):
    out = str(tmp_path / "k.ll")
    subprocess.run([build.HIPCC, "--cuda-device-only", "-S", "-emit-llvm"] + build.COMMON + build.SOURCES[source] +
                   [f"-DBHAH_PART={part}", os.path.join(build.CSRC, source), "-o", out],
                   check=True, stderr=subprocess.DEVNULL)
    ir = open(out).read()
    claims = re.findall(r"(?:load|store) <\d+ x double>[^\n]*ptr addrspace\(1\)[^\n]*?, align (\d+)", ir)
    assert claims or source != "rhs_fused.hip"
    assert all(int(a) <= 8 for a in claims), sorted(set(claims))


@pytest.mark.gpu
@pytest.mark.parametrize("ng", [3, 5])
def test_arrays_off_sixteen_bytes_give_the_same_results(ng):
    print("array alignment", ng, flush=True)
    import torch
    from paper_2505_00097_amd import capi
    from paper_2505_00097_amd import workloads as wl
    g = capi.Grid(wl.SINH_CYLINDRICAL, (33, 2, 9), (20.0,) * 3, (0.2,) * 3, nghosts=ng)
    y0 = torch.from_numpy(wl.smooth_random_state(g.n, seed=3)).cuda()
    capi.apply_bcs(g.h, y0)

    def run(off):
        def arr(like):
            t = torch.zeros(like.numel() + 1, dtype=torch.float64, device="cuda")[off:off + like.numel()].view(like.shape)
            assert t.data_ptr() % 16 == 8 * off
            return t
        y, r, ws = arr(y0), arr(y0), arr(g.workspace())
        y.copy_(y0)
        capi.bssn_rhs(g.h, y, r, diss=(0.99, 0.3))
        for step in (capi.rk4_step, capi.ssprk3_step):
            step(g.h, y, ws, 0.1 * g.dt, diss=(0.99, 0.3))
        torch.cuda.synchronize()
        return r, y

    for a, b in zip(run(0), run(1)):
        assert torch.isfinite(a).all() and torch.equal(a, b)
