"""Buffer offsets of the kernels stay inside their buffers, checked on the host
over the sizes where tiles are ragged: a read past a buffer does not show in
any result, because what it brings is not stored."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_offsets_stay_in_their_buffers(tmp_path):
    exe = str(tmp_path / "address_bounds")
    r = subprocess.run(["g++", "-O1", "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-I", os.path.join(ROOT, "include"), "-I",
                        os.path.join(ROOT, "paper_2310_03979_amd", "csrc"), "-isystem", "/opt/rocm/include",
                        os.path.join(ROOT, "tests", "host", "address_bounds.cpp"), "-o", exe], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    r = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0 and "address bounds: ok" in r.stdout, r.stdout
