"""Host memory that runs out during an assembly is an error of the call, on whichever
thread it is met, and not the end of the process."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_failed_allocations_are_errors(tmp_path):
    from paper_2306_11324_amd import build as b
    cxx = shutil.which("g++") or shutil.which("c++")
    if cxx is None:
        pytest.skip("no host compiler")
    if not os.path.exists(b.LIB):
        b.build()
    exe = str(tmp_path / "driver")
    r = subprocess.run([cxx, "-std=c++17", "-O1", "-pthread", "-I", os.path.join(ROOT, "include"), "-o", exe,
                        os.path.join(ROOT, "tests", "assembly_without_memory.cpp"), b.LIB,
                        "-Wl,-rpath," + os.path.dirname(b.LIB), "-Wl,--allow-shlib-undefined"],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-3000:]
    r = subprocess.run([exe], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, (r.returncode, r.stdout, r.stderr[-1000:])
