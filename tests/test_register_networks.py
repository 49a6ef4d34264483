"""The register-local u32 networks of csrc/bcf_device.hpp (three-input minima,
medians and maxima), compiled for the host and run on every 0-1 input of their
preconditions (``tests/sanitize/networks_check.cpp``)."""

import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1306_5076_amd", "csrc")
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")


@pytest.mark.skipif(not os.path.exists(HIPCC), reason="hipcc not installed")
def test_register_networks_on_every_01_input(tmp_path):
    exe = str(tmp_path / "networks_check")
    build = subprocess.run([HIPCC, "-x", "hip", "--offload-arch=gfx950", "--cuda-host-only", "-O1", "-std=c++17", "-I", CSRC,
                            os.path.join(ROOT, "tests", "sanitize", "networks_check.cpp"), "-o", exe],
                           stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    assert build.returncode == 0, build.stdout[-4000:]
    run = subprocess.run([exe], stdout=subprocess.PIPE, text=True, timeout=120)
    assert run.returncode == 0 and "0 failures" in run.stdout, run.stdout
