"""The compact test's table read stays in range for any A_r (CPU only: the host
compilation of the kernels' own function, with the conversion checked)."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HIPCC = "/opt/rocm/bin/hipcc"

pytestmark = pytest.mark.timeout(300)


def test_compact_bin_is_in_range(tmp_path):
    if not os.path.exists(HIPCC):
        pytest.skip("hipcc not installed")
    exe = tmp_path / "compact_bin"
    subprocess.check_call([HIPCC, "--offload-arch=gfx950", "-Xclang", "-target-feature", "-Xclang",
                           "-packed-fp32-ops", "-O1", "-std=c++17", "-Xarch_host", "-fsanitize=float-cast-overflow",
                           "-Xarch_host", "-fno-sanitize-recover=float-cast-overflow", "-I",
                           os.path.join(ROOT, "paper_2402_11354_amd", "csrc"),
                           os.path.join(ROOT, "tests", "host", "compact_bin.hip"), "-o", str(exe)],
                          stderr=subprocess.DEVNULL)
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, (r.stdout + r.stderr)[-2000:]
    assert "runtime error" not in r.stderr and "compact bin ok" in r.stdout
