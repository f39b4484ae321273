"""Work items and pieces of the row kernels (CPU only): tests/host_split.cpp, built against the
C ABI's source with host memory in the place of device memory, checks that every row is covered
once, that the pieces of a cut item meet in slots of their own, and that a re-split which runs
out of memory leaves the one in use; that branches which run out of memory leave one.  Also which rows take the modulation's FP32 series."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)


@pytest.mark.timeout(600)
def test_work_item_tables(tmp_path):
    cxx = shutil.which("g++")
    if not cxx or not os.path.isdir("/opt/rocm/include/hip"):
        pytest.skip("no host compiler or no HIP headers here")
    exe = str(tmp_path / "host_split")
    cmd = [cxx, "-std=c++17", "-O1", "-g", "-w", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
           f"-I{ROOT}/include", f"-I{ROOT}/paper_2605_26347_amd/csrc",
           os.path.join(HERE, "host_split.cpp"), "-no-pie",
           "-Wl,--unresolved-symbols=ignore-all", "-o", exe]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-4000:]
    r = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0 and "host split ok" in r.stdout, r.stdout + r.stderr
