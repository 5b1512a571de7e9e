"""The pattern analysis's index arithmetic at block positions and thread numbers beyond 2^30 and 2^31:
the functions that the kernels run, compiled for the host and called on sparse arrays
(tests/host/index_limits.cpp). No device of this size of pattern is needed, and none is touched."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_index_limits(tmp_path):
    exe = str(tmp_path / "index_limits")
    subprocess.check_call([os.environ.get("HIPCC", "/opt/rocm/bin/hipcc"), "-x", "hip", "--offload-host-only",
                           "-std=c++17", "-O1", "-I", os.path.join(ROOT, "include"),
                           "-I", os.path.join(ROOT, "paper_1912_00539_amd", "csrc"),
                           os.path.join(ROOT, "tests", "host", "index_limits.cpp"), "-o", exe])
    out = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert out.returncode == 0 and out.stdout == "OK\n", (out.returncode, out.stdout, out.stderr)
