"""Host code that the flow server and the faster kernels rest on, against plain forms of
itself: tests/sanitize/host_parts.cpp, built with g++ under AddressSanitizer and
UndefinedBehaviorSanitizer (CPU only)."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(ROOT, "paper_2607_24908_amd", "csrc")


@pytest.mark.skipif(shutil.which("g++") is None, reason="g++ not found")
def test_eliminations_and_tables(tmp_path):
    exe = str(tmp_path / "host_parts")
    b = subprocess.run(
        ["g++", "-std=c++17", "-O1", "-g", "-fsanitize=address,undefined",
         "-fno-sanitize-recover=all", "-fno-omit-frame-pointer", "-D__HIP_PLATFORM_AMD__",
         "-I/opt/rocm/include", "-I" + os.path.join(ROOT, "include"), "-I" + CSRC,
         os.path.join(HERE, "sanitize", "host_parts.cpp"), os.path.join(CSRC, "tables.cpp"),
         "-o", exe], capture_output=True, text=True, timeout=300)
    if b.returncode != 0 and "asan" in (b.stderr or "").lower():
        pytest.skip("sanitizer runtime not available: " + b.stderr[-300:])
    assert b.returncode == 0, b.stderr[-2000:]
    r = subprocess.run([exe], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0 and "host parts ok" in r.stdout, (r.stdout + r.stderr)[-4000:]
