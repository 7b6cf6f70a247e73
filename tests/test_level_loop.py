"""The host's level loop (``run_levels``) without a GPU: the library's host
sources linked with a replay of the level kernels' control protocol, over
frontiers on both sides of every size at which a launch rule changes."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1708_01159_amd", "csrc")


@pytest.mark.skipif(shutil.which("g++") is None, reason="g++ not found")
def test_every_search_reads_all_its_levels(tmp_path):
    exe = str(tmp_path / "level_loop")
    r = subprocess.run(["g++", "-std=c++17", "-O1", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
                        "-I" + os.path.join(ROOT, "include"), os.path.join(ROOT, "tests", "host", "level_loop.cpp"),
                        os.path.join(CSRC, "gsw_bfs.cpp"), os.path.join(CSRC, "gsw_core.cpp"), "-o", exe],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-3000:]
    r = subprocess.run([exe], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0 and r.stdout.strip() == "ok", r.stdout + r.stderr[-4000:]
