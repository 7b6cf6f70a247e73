"""The host's level loop (``run_levels``) without a GPU: the library's host
sources linked with a replay of the level kernels' control protocol, over
frontiers on both sides of every size at which a launch rule changes; and the
host memory that gsw_bfs_noalloc's records go to."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1708_01159_amd", "csrc")
CLANG = "/opt/rocm/llvm/bin/clang++"


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


@pytest.mark.skipif(not os.path.exists(CLANG), reason="ROCm toolchain not found")
def test_noalloc_records_with_and_without_mapped_memory(tmp_path):
    flags = ["-std=c++17", "-O1", "-g", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
             "-I" + os.path.join(ROOT, "include")]
    obj = str(tmp_path / "noalloc.o")
    r = subprocess.run([CLANG, "-x", "hip", "--offload-host-only", "--offload-arch=gfx950"] + flags
                       + ["-c", os.path.join(CSRC, "gsw_noalloc.hip"), "-o", obj], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-3000:]
    exe = str(tmp_path / "noalloc_ring")
    # (the device code that the object names is not there and never used)
    r = subprocess.run([CLANG] + flags + [os.path.join(ROOT, "tests", "host", "noalloc_ring.cpp"),
                                          os.path.join(CSRC, "gsw_bfs.cpp"), os.path.join(CSRC, "gsw_core.cpp"), obj,
                                          "-Wl,--unresolved-symbols=ignore-in-object-files", "-o", exe],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-3000:]
    r = subprocess.run([exe], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0 and r.stdout.strip() == "ok", r.stdout + r.stderr[-4000:]
