"""The short sine and cosine of the kernels, compiled for the host: accuracy over the
stated ranges, bounded beyond them, NaN where the argument is not finite."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_ranges_and_values_that_are_not_finite(tmp_path):
    from paper_2306_11324_amd import build as b
    try:
        hipcc = b.hipcc()
    except RuntimeError:
        pytest.skip("no hipcc")
    exe = str(tmp_path / "sincos")
    r = subprocess.run([hipcc, f"--offload-arch={b.ARCH}", "--offload-host-only", "-O2", "-std=c++17",
                        "-I", os.path.join(ROOT, "include"),
                        "-I", os.path.join(ROOT, "paper_2306_11324_amd", "csrc"), "-o", exe,
                        os.path.join(ROOT, "tests", "short_sincos.hip")], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-3000:]
    out = [ln.split() for ln in subprocess.run([exe], capture_output=True, text=True, check=True).stdout.splitlines()]
    for bits, worst, largest in out[:-4]:
        # two roundings of values up to 1 (and, where |r| may pass pi/4, the polynomials' growth)
        if int(bits) <= 48:
            assert float(worst) <= 2.5e-16, (bits, worst)
        elif int(bits) <= 50:
            assert float(worst) <= 1e-15, (bits, worst)
        assert float(largest) <= 1.0 + 1e-12, (bits, largest)
    assert out[-4:-1] == [["1", "1"]] * 3
    assert out[-1] == ["0", "1"]
