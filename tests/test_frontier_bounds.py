"""Where the level kernels read their input arrays, against the memory that an
external workspace's call carves for them (no GPU): the host's own carve at the
least memory a call accepts, its own choice of levels, every depth up to 26,
first calls and later ones whose first level follows the frontier."""
import os
import shutil
import subprocess

from paper_2311_02573_amd import build, gt

HERE = os.path.dirname(os.path.abspath(__file__))


def test_level_input_reads_stay_inside_the_carved_frontier(tmp_path):
    exe = str(tmp_path / "frontier_bounds")
    hipcc = shutil.which("hipcc") or build.HIPCC
    # (host code only; the choice of levels that the kernels' files hold comes
    # from the built library)
    lib = os.path.dirname(gt.LIB_PATH)
    cmd = [hipcc, "-x", "hip", "--offload-host-only", "-O1", "-std=c++17", "-fPIC", "-w",
           "-I", os.path.join(build.ROOT, "include"), "-I", build.CSRC, "-c",
           os.path.join(HERE, "native", "frontier_bounds.cpp"), "-o", exe + ".o"]
    subprocess.run(cmd, check=True, timeout=300)
    subprocess.run([hipcc, exe + ".o", "-o", exe, gt.LIB_PATH, "-Wl,-rpath," + lib], check=True, timeout=300)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stderr
    cases, plain, beyond = map(int, r.stdout.split())
    # the slot's plain index leaves the memory in some of these: they cover it
    assert cases > 10000 and plain > 100
    assert beyond == 0
