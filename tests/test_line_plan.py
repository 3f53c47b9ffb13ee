"""Host-only check of the windows of the 1D kernel of many steps per launch
(tests/native/line_bounds.hip)."""
import os
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))


def test_line_windows_cover_the_mesh_and_stay_in_bounds(tmp_path):
    hipcc = "/opt/rocm/bin/hipcc"
    if not os.path.exists(hipcc):
        pytest.skip("hipcc not available")
    exe = str(tmp_path / "line_bounds")
    subprocess.run([hipcc, "--offload-host-only", "-O1", "-std=c++17", "-fconstexpr-steps=100000000",
                    os.path.join(HERE, "native", "line_bounds.hip"), "-o", exe], check=True, capture_output=True)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stdout + r.stderr
