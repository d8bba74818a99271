"""The pool of kept device memory under memory pressure, against a device that the test program plays."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_kept_memory_is_given_back_to_every_allocation_that_fails(tmp_path):
    exe = str(tmp_path / "device_keep_test")
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
                           "-I", os.path.join(ROOT, "paper_2504_06443_amd", "csrc"), "-o", exe,
                           os.path.join(ROOT, "tests", "host", "device_keep_test.cpp")])
    run = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    assert run.returncode == 0, run.stdout + run.stderr
