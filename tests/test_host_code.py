"""Host code of the library that needs no GPU, compiled with g++: the pool of kept device memory under
memory pressure (against a device that the test program plays), and the LDS layouts of the plan."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.mark.parametrize("program", ["device_keep_test", "panel_layout_test"])
def test_host_program(program, tmp_path):
    exe = str(tmp_path / program)
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
                           "-I", os.path.join(ROOT, "paper_2504_06443_amd", "csrc"), "-o", exe,
                           os.path.join(ROOT, "tests", "host", program + ".cpp")])
    run = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    assert run.returncode == 0, run.stdout + run.stderr
