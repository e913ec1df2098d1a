"""AddressSanitizer and UndefinedBehaviorSanitizer build of the stencil boxes
of the particle kernels (csrc/amrmg_box.hpp, host and device code), driven by
tests/native/box_sanitize.cpp: no signed overflow, also for the box of no
particle.  Host code only."""
import os

from test_sanitizers import NATIVE, ROOT, SAN, run


def test_boxes_under_sanitizers(tmp_path):
    csrc = os.path.join(ROOT, "paper_1812_03689_amd", "csrc")
    out = run(["g++", "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-Wno-unknown-pragmas", "-I" + csrc, "-isystem", "/opt/rocm/include"] + SAN +
              [os.path.join(NATIVE, "box_sanitize.cpp")], str(tmp_path / "box_sanitize"))
    assert "box sanitize ok" in out
