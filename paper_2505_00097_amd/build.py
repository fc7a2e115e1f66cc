"""Build the HIP library libbhah.so (gfx950) in-tree.

Each source is compiled with hipcc for gfx950; the right-hand-side and
constraint units also get -fno-signed-zeros -ffinite-math-only so that
structurally zero reference-metric terms fold away (no reassociation is
enabled). They fuse multiply-adds only where the source writes them in one
expression (-ffp-contract=on), so that every kernel that inlines the same code
rounds alike whatever the compiler makes of its surroundings, and are compiled
in parts (one kernel variant each), in parallel.
"""
import concurrent.futures as cf
import os
import subprocess

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
OBJ = os.path.join(HERE, "_build")
LIB = os.path.join(HERE, "libbhah.so")
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")

COMMON = ["-O3", "-fPIC", "-std=c++17", "-Wall", "-Wno-unused-function"]
ARCH = ["--offload-arch=gfx950", "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops"]
DEVICE = ARCH + ["-ffp-contract=fast"]
STENCIL = ARCH + ["-ffp-contract=on", "-fno-signed-zeros", "-ffinite-math-only"]
SOURCES = {
    "rhs_fused.hip": STENCIL,
    "hamiltonian.hip": STENCIL,
    "misc.hip": DEVICE,
    "probe.hip": DEVICE,
    "grid.cpp": [],
    "capi.cpp": [],
    "engine.cpp": [],
    "batch.cpp": [],
    "server.cpp": [],
}
PARTS = {"rhs_fused.hip": 12, "hamiltonian.hip": 12}  # compiled once per part, -DBHAH_PART=0 ..


def _compile(name, extra, part, verbose):
    src = os.path.join(CSRC, name)
    obj = os.path.join(OBJ, f"{name}.{part}.o" if part is not None else name + ".o")
    cmd = [HIPCC] + COMMON + extra + ([f"-DBHAH_PART={part}"] if part is not None else []) + ["-c", src, "-o", obj]
    if verbose:
        print(" ".join(cmd), flush=True)
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"compile failed: {name} {part}\n{r.stdout}\n{r.stderr}")
    return obj


def build(verbose: bool = False) -> str:
    os.makedirs(OBJ, exist_ok=True)
    with cf.ThreadPoolExecutor(max_workers=min(8, os.cpu_count() or 1)) as ex:
        units = [(n, e, p) for n, e in SOURCES.items() for p in (range(PARTS[n]) if n in PARTS else [None])]
        futs = [ex.submit(_compile, n, e, p, verbose) for n, e, p in units]
        objs = [f.result() for f in futs]
    cmd = [HIPCC, "-shared", "-fPIC", "--offload-arch=gfx950", "-o", LIB + ".tmp"] + objs
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.run(cmd, check=True)
    os.replace(LIB + ".tmp", LIB)
    return LIB


if __name__ == "__main__":
    print(build(verbose=True))
