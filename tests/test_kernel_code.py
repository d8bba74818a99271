"""Loads that a kernel's design keeps in flight, in the code that hipcc makes for gfx950: the compiler may
sink a load down to its use, which no result shows."""
import os
import re
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def product_kernels(tmp_path_factory):
    from paper_2504_06443_amd import build
    out = str(tmp_path_factory.mktemp("asm") / "exec_kernels.s")
    flags = [f for f in build.FLAGS if f not in ("-shared", "-fPIC")]
    subprocess.check_call([os.environ.get("HIPCC", "/opt/rocm/bin/hipcc"), *flags, "-S", "--offload-device-only", "-o", out,
                           os.path.join(build.CSRC, "exec_kernels.hip")], stderr=subprocess.DEVNULL)
    with open(out) as f:
        return f.read()


def instructions(code, kernel):
    body = re.search(r"^_ZN4spmm\S*%s\S*:.*?s_endpgm" % kernel, code, re.M | re.S)[0]
    return [line.split(";")[0].strip() for line in body.splitlines()]


def test_merge_loads_a_round_of_parts_at_a_time(product_kernels):
    longest = run = 0
    for i in instructions(product_kernels, "k_merge"):
        if i.startswith("global_load_dwordx4"):
            run += 1
            longest = max(longest, run)
        elif i.startswith(("s_cbranch", "s_branch", ".LBB")) or re.match(r"s_waitcnt.*vmcnt\(0\)", i):
            run = 0
    assert longest >= 16
