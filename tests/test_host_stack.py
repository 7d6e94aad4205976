"""The library's host code leaves its caller's stack alone (CPU only): no function of
the C interface's sources has a frame above 16 KB, so that a thread of the smallest
usual stack can call it."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1607_04069_amd", "csrc")
HIPCC = "/opt/rocm/bin/hipcc"


@pytest.mark.parametrize("source", ["capi.hip", "tpm_kernels.hip", "pic_kernels.hip"])
def test_frames_are_small(source):
    if not os.path.exists(HIPCC):
        pytest.skip("no hipcc")
    r = subprocess.run([HIPCC, "-O3", "-std=c++17", "-fPIC", "--offload-arch=gfx950", "--offload-host-only",
                        "-Wframe-larger-than=16384", "-I", os.path.join(ROOT, "include"), "-I", CSRC, "-c",
                        os.path.join(CSRC, source), "-o", os.devnull], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    assert "stack frame size" not in r.stderr, r.stderr
