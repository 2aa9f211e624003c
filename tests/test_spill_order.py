"""A spilled query's visited test comes after the bits it looks for: in the
compiled search kernels every read of the bitmap waits until the atomics
before it, which set the last survivors' bits, are complete (CPU only: the
gfx950 assembly of two instantiations, compiled here)."""
import os
import re
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HIPCC = "/opt/rocm/bin/hipcc"

pytestmark = pytest.mark.timeout(300)


@pytest.mark.parametrize("inst", ["8, 0, true", "8, 0, false"])
def test_bitmap_reads_wait_for_the_bits(tmp_path, inst):
    if not os.path.exists(HIPCC):
        pytest.skip("hipcc not installed")
    src = tmp_path / "one.hip"
    src.write_text('#include "k_search.hpp"\n'
                   f"template __global__ void peos::k_search<{inst}>(peos::SearchArgs);\n")
    asm = tmp_path / "one.s"
    subprocess.check_call([HIPCC, "--offload-arch=gfx950", "-O3", "-std=c++17", "-Xclang", "-target-feature",
                           "-Xclang", "-packed-fp32-ops", "--cuda-device-only", "-S", "-I",
                           os.path.join(ROOT, "paper_2402_11354_amd", "csrc"), str(src), "-o", str(asm)],
                          stderr=subprocess.DEVNULL)
    text = asm.read_text()
    body = text[text.index("k_search"):].splitlines()
    # the bitmap is read by the only device-scope loads of the kernel
    reads = [i for i, s in enumerate(body) if re.search(r"global_load_dword\s.*\bsc1\b", s)]
    sets = [i for i, s in enumerate(body) if "global_atomic_or" in s]
    assert reads and sets
    for r in reads:
        before = [s for s in sets if s < r]
        assert before
        assert any(re.search(r"s_waitcnt\s.*vmcnt\(0\)", s) for s in body[before[-1]:r])
