"""Host-side parts of the library that the GPU tests cannot check safely, run
without a GPU under the address and undefined-behaviour sanitizers: the rows
that the inverse row kernel reads, the FFT lengths that a geometry is padded
to, and the batched runtime's handling of buffers, streams and graphs."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1102_3069_amd", "csrc")
OBJ = os.path.join(ROOT, "paper_1102_3069_amd", "_build")
HIPCC = os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "bin", "hipcc")

pytestmark = pytest.mark.skipif(not os.path.exists(HIPCC), reason="no hipcc")


def newest(*dirs):
    return max(os.path.getmtime(os.path.join(d, f)) for d in dirs for f in os.listdir(d) if not f.endswith(".pyc"))


def build(name, *extra):
    """tests/host/<name>.hip with the sanitizers on the host side."""
    host = os.path.join(ROOT, "tests", "host")
    out = os.path.join(OBJ, name + "_sanitized")
    os.makedirs(OBJ, exist_ok=True)
    if not os.path.exists(out) or os.path.getmtime(out) < newest(host, CSRC, os.path.join(ROOT, "include")):
        cmd = [HIPCC, "--offload-arch=gfx950", "-O1", "-g", "-std=c++17",
               "-Xarch_host", "-fsanitize=address", "-Xarch_host", "-fsanitize=undefined",
               "-Xarch_host", "-fno-sanitize-recover=all",
               "-I", os.path.join(ROOT, "include"), "-I", CSRC, os.path.join(host, name + ".hip"), *extra, "-o", out]
        r = subprocess.run(cmd, capture_output=True, text=True)
        assert r.returncode == 0, r.stderr[-4000:]
    return out


def run(out, *args):
    r = subprocess.run([out, *args], capture_output=True, text=True, timeout=300,
                       env=dict(os.environ, ASAN_OPTIONS="detect_leaks=0"))
    assert r.returncode == 0, r.stdout[-2000:] + r.stderr[-4000:]
    return r.stdout


def test_staged_rows_stay_inside_the_film():
    assert "staged rows ok" in run(build("host_rows"))


def library():
    """Link arguments for the library as it is built."""
    pkg = os.path.dirname(OBJ)
    if not os.path.exists(os.path.join(pkg, "libllg.so")):
        import __graft_entry__
        __graft_entry__.build()
    rocm = os.path.dirname(os.path.dirname(HIPCC))
    return ["-L" + pkg, "-l:libllg.so", "-Wl,-rpath," + pkg, "-L" + os.path.join(rocm, "lib"), "-lrocprofiler-sdk-roctx"]


def test_padded_lengths():
    assert "padding ok" in run(build("host_padding", *library()))


def test_batches_run_to_their_end_again_and_again():
    """Three batches of 64 uneven films, set anew and run to t_end 40 times, with
    fixed steps, tuning and re-creation in between, on a stand-in for the HIP
    runtime: no access outside an allocation, no use after a release, no broken
    rule of captures, every resource given back."""
    assert "batch ok" in run(build("host_batch", *library()))
