"""CPU test of the staged copies to host memory (hostcopy.cpp): two devices in
one thread, sizes around the staged and the threaded copy, and the rings freed
with the last context.  Compiled as host code with the runtime's calls defined
by the test."""
import os
import subprocess

from paper_2606_22180_amd import build

HERE = os.path.dirname(os.path.abspath(__file__))


def test_copies_of_two_devices(tmp_path):
    exe = str(tmp_path / "hostcopy_devices")
    subprocess.run([build.hipcc(), "-x", "hip", "--offload-host-only", "-O1", "-std=c++17",
                    "-Wno-unused-result", "-I", os.path.join(build.ROOT, "include"),
                    "-I", build.CSRC, os.path.join(HERE, "native", "hostcopy_devices.cpp"),
                    "-o", exe, "-lpthread"], check=True, capture_output=True, text=True)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0 and r.stdout == "ok\n", (r.returncode, r.stderr)
