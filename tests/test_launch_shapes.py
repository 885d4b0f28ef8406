"""The launch shapes that the entry points choose (csrc/cx_launch.hpp): rules that no result shows, checked by the
compiler.  CPU only."""
import os
import subprocess

from paper_2012_15198_amd import build

HERE = os.path.dirname(os.path.abspath(__file__))


def test_launch_shapes():
    out = subprocess.run([os.environ.get("HIPCC", "/opt/rocm/bin/hipcc"), *build.HIPCC_FLAGS, "--cuda-host-only", "-fsyntax-only",
                          "-I", os.path.join(build.ROOT, "include"), "-I", build.CSRC,
                          os.path.join(HERE, "host", "launch_shapes_check.hip")], capture_output=True, text=True, timeout=300)
    assert out.returncode == 0, out.stderr[-6000:]
