"""The C entry that allocates host memory returns ABILU_ENOMEM where there is none: a C++ program whose
operator new fails (tests/host/no_memory.cpp), run as a child process."""
import os
import subprocess

from paper_1912_00539_amd import build

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_no_host_memory(tmp_path):
    exe, lib = str(tmp_path / "no_memory"), build.OUTDIR
    tl = build.torch_lib_dir() or "/opt/rocm/lib"
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-I", build.INCLUDE,
                           os.path.join(ROOT, "tests", "host", "no_memory.cpp"), "-o", exe, f"-L{lib}", "-labilu",
                           f"-Wl,-rpath,{lib}", f"-L{tl}", f"-Wl,-rpath,{tl}", "-Wl,--allow-shlib-undefined"])
    out = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    assert out.returncode == 0 and out.stdout == "OK\n", (out.returncode, out.stdout, out.stderr)
