"""Builds the HIP library libllg.so in-tree for gfx950 with hipcc: each
source is compiled to an object in parallel (the 2D kernels in several
parts), then they are linked."""
import os
import subprocess
import sys
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
OBJ = os.path.join(HERE, "_build")
LIB = os.path.join(HERE, "libllg.so")
SOURCES = ["fast2d.hip", "kernels.hip", "fast3d.hip", "tensor.hip", "solver.hip", "batch.hip", "surrogate.hip"]
# sources compiled once per part of their kernel variants: (macro, parts)
PARTS = {"fast2d.hip": ("FAST2D_PART", 5)}


def hipcc():
    rocm = os.environ.get("ROCM_PATH", "/opt/rocm")
    return os.path.join(rocm, "bin", "hipcc")


FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC",
    # packed-FP32 instructions off: hand-written kernels use scalar FP32
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-I", os.path.join(ROOT, "include"), "-I", CSRC,
]


def _compile(unit, verbose):
    src, part = unit
    obj = os.path.join(OBJ, os.path.splitext(src)[0] + ("" if part is None else f"_{part}") + ".o")
    define = [] if part is None else [f"-D{PARTS[src][0]}={part}"]
    cmd = [hipcc()] + FLAGS + define + ["-c", os.path.join(CSRC, src), "-o", obj]
    if verbose:
        print(" ".join(cmd), flush=True)
    r = subprocess.run(cmd, capture_output=True, text=True)
    noise = "is not a recognized feature for this target"
    err = "\n".join(l for l in r.stderr.splitlines() if noise not in l)
    if r.returncode != 0:
        raise RuntimeError(f"hipcc failed on {src}:\n{err}")
    if err.strip() and verbose:
        print(err, flush=True)
    return obj


def build(verbose=True):
    os.makedirs(OBJ, exist_ok=True)
    units = [(src, part) for src in SOURCES for part in (range(PARTS[src][1]) if src in PARTS else (None,))]
    jobs = min(len(units), max(1, min(8, os.cpu_count() or 1)))
    with ThreadPoolExecutor(jobs) as ex:
        objs = list(ex.map(lambda u: _compile(u, verbose), units))
    tmp = LIB + ".tmp"
    rocm = os.environ.get("ROCM_PATH", "/opt/rocm")
    # roctx ranges around the API calls (rocprofv3 --marker-trace)
    libs = ["-L" + os.path.join(rocm, "lib"), "-Wl,-rpath," + os.path.join(rocm, "lib"), "-lrocprofiler-sdk-roctx"]
    cmd = [hipcc(), "--offload-arch=gfx950", "-shared", "-fPIC", "-o", tmp] + objs + libs
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.run(cmd, check=True)
    os.replace(tmp, LIB)
    return LIB


if __name__ == "__main__":
    build()
    sys.exit(0)
