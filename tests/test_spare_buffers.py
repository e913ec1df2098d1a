"""Device buffers that find no room have the particle records given back
(csrc/amrmg_state.hpp), on the CPU with stand-ins for the runtime's memory
functions (tests/native/spare_buffers.cpp)."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_records_are_given_back(tmp_path):
    exe = str(tmp_path / "spare_buffers")
    inc = [os.path.join(ROOT, "include"), os.path.join(ROOT, "paper_1812_03689_amd", "csrc")]
    b = subprocess.run(["g++", "-std=c++17", "-O1", "-D__HIP_PLATFORM_AMD__"] + ["-I" + i for i in inc] +
                       ["-isystem", "/opt/rocm/include", os.path.join(ROOT, "tests", "native", "spare_buffers.cpp"),
                        "-o", exe], capture_output=True, text=True)
    assert b.returncode == 0, b.stderr
    r = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0 and "spare buffers ok" in r.stdout, r.stdout + r.stderr
