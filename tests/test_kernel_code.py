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


def test_narrow_tile_enters_its_loop_with_the_ring_full(product_kernels):
    """Four steps of two loads are in flight at the head of the check-free loop, and the loop begins with
    three more: the first operand waits for none of the eight youngest."""
    code = instructions(product_kernels, "k_spmm_mfma_fastILi1ELb0E")
    heads = {i[:-1]: n for n, i in enumerate(code) if i.startswith(".LBB")}
    loops = [code[heads[i.split()[1]]:n] for n, i in enumerate(code)
             if i.startswith("s_cbranch") and heads.get(i.split()[1], n) < n]
    steady = [body for body in loops if sum(i.startswith("v_mfma") for i in body) == 8
              and not any(i.startswith("s_cbranch") for i in body)]
    assert len(steady) == 1
    waits = [int(m[1]) for m in (re.search(r"vmcnt\((\d+)\)", i) for i in steady[0]) if m]
    assert waits[0] >= 8
