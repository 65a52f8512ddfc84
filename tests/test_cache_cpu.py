"""The library's cache of freed device buffers on the CPU, over a stub of the
runtime's allocator: sizes, limits, refusals, and one thread freeing and
another setting the limit while a third allocates, under ThreadSanitizer and
under AddressSanitizer (host code only)."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2310_15668_amd", "csrc")

pytestmark = pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")


@pytest.mark.parametrize("sanitizer", ["thread", "address,undefined"])
def test_cache(tmp_path, sanitizer):
    exe = str(tmp_path / "cache")
    res = subprocess.run(["g++", "-std=c++17", f"-fsanitize={sanitizer}", "-g", "-O1", "-pthread",
                          "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", "-I", os.path.join(ROOT, "include"),
                          "-I", CSRC, "-o", exe, os.path.join(CSRC, "cache.cpp"),
                          os.path.join(ROOT, "tests", "sanitize", "cache_driver.cpp")], capture_output=True, text=True)
    assert res.returncode == 0, res.stderr
    res = subprocess.run([exe], capture_output=True, text=True, timeout=300)
    assert res.returncode == 0, res.stdout + res.stderr
    assert "cache ok" in res.stdout and "Sanitizer" not in res.stderr, res.stderr
