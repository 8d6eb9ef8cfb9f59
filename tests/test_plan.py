"""Host check of the planned sizes (scratch, workspaces, launches): the check
program tests/plan_check.cpp is built for the host with hipcc from the library's
own headers; no GPU is used."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_planned_sizes_cover_what_is_written(tmp_path):
    hipcc = shutil.which("hipcc") or ("/opt/rocm/bin/hipcc" if os.path.exists("/opt/rocm/bin/hipcc") else None)
    if hipcc is None:
        pytest.skip("hipcc not found")
    exe = str(tmp_path / "plan_check")
    r = subprocess.run([hipcc, "-O1", "-std=c++17", "--offload-arch=gfx950",
                        "-I", os.path.join(ROOT, "paper_1909_04631_amd", "csrc"),
                        "-I", os.path.join(ROOT, "include"),
                        os.path.join(ROOT, "tests", "plan_check.cpp"), "-o", exe],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-2000:]
    out = subprocess.run([exe], capture_output=True, text=True)
    print(out.stdout)
    assert out.returncode == 0 and out.stdout.strip().endswith("ok"), out.stdout
