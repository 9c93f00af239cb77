"""The pool of freed device blocks (csrc/gt_block_pool.h) over a made-up device:
reuse, its bounds, and what leaves when (no GPU)."""
import os
import shutil
import subprocess

from paper_2311_02573_amd import build

HERE = os.path.dirname(os.path.abspath(__file__))


def test_block_pool(tmp_path):
    exe = str(tmp_path / "block_pool")
    subprocess.run([shutil.which("g++") or "c++", "-std=c++17", "-O1", "-Wall", "-pthread", "-I", build.CSRC,
                    os.path.join(HERE, "native", "block_pool.cpp"), "-o", exe], check=True, timeout=300)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0 and r.stdout.endswith("done\n"), r.stdout + r.stderr
