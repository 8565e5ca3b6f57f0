"""What a call that fails half-way leaves behind, on the host alone: the library's host code linked against
launchers that only count, one of which fails (tests/host/failed_call.hip)."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_rows_after_a_failed_call(tmp_path):
    from paper_1810_08313_amd import build
    hipcc = build.HIPCC if os.path.exists(build.HIPCC) else shutil.which("hipcc")
    if not hipcc:
        pytest.skip("hipcc not available")
    exe = str(tmp_path / "failed_call")
    flags = [f for f in build.FLAGS if not f.startswith("--offload-arch")]
    subprocess.run([hipcc, *flags, "--offload-host-only", os.path.join(build.CSRC, "lc_api.hip"),
                    os.path.join(ROOT, "tests", "host", "failed_call.hip"), "-o", exe], check=True, timeout=300)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, r.stdout
