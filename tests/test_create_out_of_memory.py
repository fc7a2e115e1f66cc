"""bhah_grid_create where the host has no memory for the grid's lists: the call
returns BHAH_ENOMEM with a message; no C++ exception crosses the C boundary.
(In a process of its own with a bounded address space; no GPU needed, the lists
are built before the first device call.)"""
import subprocess
import sys

CODE = """
import ctypes, resource
from paper_2505_00097_amd import capi
lib = capi.lib()
used = int(open("/proc/self/statm").read().split()[0]) * resource.getpagesize()
resource.setrlimit(resource.RLIMIT_AS, (used + (64 << 20),) * 2)
p = capi.GridParams(0, (ctypes.c_int * 3)(200, 300, 300), 3, (ctypes.c_double * 3)(10, 10, 10),
                    (ctypes.c_double * 3)(.2, .2, .2), 0.5, 0)
h = ctypes.c_void_p()
rc = lib.bhah_grid_create(ctypes.byref(p), ctypes.byref(h))
print(rc, h.value, lib.bhah_last_error().decode())
"""


def test_grid_create_reports_a_lack_of_host_memory():
    r = subprocess.run([sys.executable, "-c", CODE], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, (r.returncode, r.stderr[-500:])
    rc, handle, msg = r.stdout.split(maxsplit=2)
    assert (rc, handle) == ("-3", "None") and "bhah_grid_create" in msg, r.stdout
