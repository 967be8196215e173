"""The sparse outlier operand of the dual family's matrix kernels decodes to
the packed codes for every position (1:8) and pair of positions (2:8).  The
function is the kernels' own header, compiled for the host by hipcc; the
check runs on the CPU."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)


def _hipcc():
    for p in (os.environ.get("HIPCC"), "/opt/rocm/bin/hipcc", shutil.which("hipcc")):
        if p and os.path.exists(p):
            return p
    pytest.skip("hipcc not found")


def test_sparse_outliers_decode_to_the_packed_codes(tmp_path):
    exe = str(tmp_path / "dual_frag")
    cmd = [_hipcc(), "-O2", "-std=c++17", "--offload-arch=gfx950", "-I" + os.path.join(ROOT, "include"),
           "-I" + os.path.join(ROOT, "paper_2406_13868_amd", "csrc"), os.path.join(HERE, "host", "dual_frag.hip"),
           "-o", exe]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    r = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0 and "dual fragments ok" in r.stdout, r.stdout + r.stderr
