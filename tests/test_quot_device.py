"""The quotient that the kernels take with the divisor's reciprocal (quot_rn), compiled
for the host from the library's header, against the division rounded once.  Quotients
below 2^-120, zeros, subnormals and infinities included."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_quotient_of_the_kernels(tmp_path):
    hipcc = shutil.which("hipcc") or ("/opt/rocm/bin/hipcc" if os.path.exists("/opt/rocm/bin/hipcc") else None)
    if hipcc is None:
        pytest.skip("hipcc not found")
    exe = str(tmp_path / "quot_check")
    r = subprocess.run([hipcc, "-O2", "-std=c++17", "-ffp-contract=off", "--offload-arch=gfx950",
                        "-I", os.path.join(ROOT, "paper_1909_04631_amd", "csrc"),
                        os.path.join(ROOT, "tests", "quot_check.cpp"), "-o", exe],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-2000:]
    out = subprocess.run([exe], capture_output=True, text=True)
    print(out.stdout)
    assert out.returncode == 0 and out.stdout.strip().endswith("ok"), out.stdout
