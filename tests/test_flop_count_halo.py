"""The FLOP figure leaves out the derivatives at the halo points of a tile's
patch, which are no terms of the equations and which a finer tiling would form
more of: it equals the count of a copy of the source in which those sums are
replaced by a value, compiled here (no GPU needed)."""
import os
import shutil
import subprocess

import pytest

from paper_2505_00097_amd import build, count_flops

# the sums at halo points, and what stands in their place in the copy
HALO = [("S.put_e(t, s[t][E].d1, d1_sum<R>(vh[t]))", "S.put_e(t, s[t][E].d1, vh[t][0])"),
        ("S.put_e(0, s[E].d1, d1_sum<R>(vh))", "S.put_e(0, s[E].d1, vh[0])"),
        ("put_halo(r, d1_sum<R>(h.lo), d1_sum<R>(h.hi))", "put_halo(r, h.lo[0], h.hi[0])"),
        ("dP[2 * r] = d1_sum<R>(h[r].lo)", "dP[2 * r] = h[r].lo[0]"),
        ("dP[2 * r + 1] = d1_sum<R>(h[r].hi)", "dP[2 * r + 1] = h[r].hi[0]")]


def _ir(csrc, part, out):
    subprocess.run([build.HIPCC, "--cuda-device-only", "-S", "-emit-llvm"] + build.COMMON +
                   build.SOURCES["rhs_fused.hip"] + [f"-DBHAH_PART={part}", os.path.join(csrc, "rhs_fused.hip"), "-o",
                                                     out], check=True, stderr=subprocess.DEVNULL)
    return open(out).read()


@pytest.mark.parametrize("part", [0, 3, 8, 11])  # both orders, with two phi planes and more
def test_flops_leave_out_the_halo(tmp_path, part):
    csrc = str(tmp_path / "p" / "csrc")
    shutil.copytree(build.CSRC, csrc)
    shutil.copytree(os.path.join(os.path.dirname(os.path.dirname(build.CSRC)), "include"), str(tmp_path / "include"))
    path = os.path.join(csrc, "rhs_stencil.h")
    text = open(path).read()
    for old, new in HALO:
        assert text.count(old) == 1, old
        text = text.replace(old, new)
    open(path, "w").write(text)
    case, ng = (part // 2 % 3, part % 2 == 1), 5 if part >= 6 else 3
    ir, without = _ir(build.CSRC, part, str(tmp_path / "a.ll")), _ir(csrc, part, str(tmp_path / "b.ll"))
    for ko in (False, True):
        figure = count_flops.count(ir, dissipation=ko, nghosts=ng)[case]
        rest = count_flops.count(without, dissipation=ko, nghosts=ng)[case] + count_flops.HALO_SHARE[(ng, case[1])]
        assert figure == rest, (ko, figure, rest)
