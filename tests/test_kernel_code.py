"""What no result shows, in the code that hipcc makes for gfx950: loads that a kernel's design keeps in flight
(the compiler may sink a load down to its use), and waits between what a kernel writes and the signal that it
has."""
import os
import re
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def compiled(source, directory):
    from paper_2504_06443_amd import build
    out = str(directory / (source + ".s"))
    flags = [f for f in build.FLAGS if f not in ("-shared", "-fPIC")]
    subprocess.check_call([os.environ.get("HIPCC", "/opt/rocm/bin/hipcc"), *flags, "-S", "--offload-device-only", "-o", out,
                           os.path.join(build.CSRC, source)], stderr=subprocess.DEVNULL)
    with open(out) as f:
        return f.read()


@pytest.fixture(scope="module")
def product_kernels(tmp_path_factory):
    return compiled("exec_kernels.hip", tmp_path_factory.mktemp("asm"))


@pytest.fixture(scope="module")
def plan_kernels(tmp_path_factory):
    return compiled("plan_kernels.hip", tmp_path_factory.mktemp("asm"))


def instructions(code, kernel):
    bodies = re.findall(r"^_ZN4spmm\S*%s\S*:.*?^\.Lfunc_end" % kernel, code, re.M | re.S)
    assert len(bodies) == 1, "%d functions are named like %s" % (len(bodies), kernel)
    return [line.split(";")[0].strip() for line in bodies[0].splitlines()]


def test_merge_loads_a_round_of_parts_at_a_time(product_kernels):
    longest = run = 0
    for i in instructions(product_kernels, "k_merge"):
        if i.startswith("global_load_dwordx4"):
            run += 1
            longest = max(longest, run)
        elif i.startswith(("s_cbranch", "s_branch", ".LBB")) or re.match(r"s_waitcnt.*vmcnt\(0\)", i):
            run = 0
    assert longest >= 16


@pytest.mark.parametrize("waves", [4, 1])              # a workgroup
def test_narrow_tile_enters_its_loop_with_the_ring_full(product_kernels, waves):
    """Four steps of two loads are in flight at the head of the check-free loop, and the loop begins with
    three more: the first operand waits for none of the eight youngest."""
    code = instructions(product_kernels, "k_spmm_mfma_fastILi1ELb0ELb0ELi%dE" % waves)
    heads = {i[:-1]: n for n, i in enumerate(code) if i.startswith(".LBB")}
    loops = [code[heads[i.split()[1]]:n] for n, i in enumerate(code)
             if i.startswith("s_cbranch") and heads.get(i.split()[1], n) < n]
    steady = [body for body in loops if sum(i.startswith("v_mfma") for i in body) == 8
              and not any(i.startswith("s_cbranch") for i in body)]
    assert len(steady) == 1
    waits = [int(m[1]) for m in (re.search(r"vmcnt\((\d+)\)", i) for i in steady[0]) if m]
    assert waits[0] >= 8


def test_plan_stats_signals_behind_what_every_wavefront_wrote(plan_kernels):
    """The thread that counts its workgroup as ended (an atomic that returns the count) and the one that sets
    the host's flag (the last store) do so behind a barrier; each wavefront comes to that barrier with nothing
    of its own under way: the wait stands in the barrier's own basic block, so no branch leads past it."""
    code = instructions(plan_kernels, "k_plan_stats")
    counted = max(n for n, i in enumerate(code) if i.startswith("global_atomic_add") and i.endswith("sc0"))
    flagged = max(n for n, i in enumerate(code) if i.startswith(("global_store", "flat_store")))
    assert counted < flagged
    barriers = []
    for signal in (counted, flagged):
        at = max(n for n in range(signal) if code[n] == "s_barrier")
        barriers.append(at)
        waited = False
        for i in reversed(code[:at]):
            if re.match(r"s_waitcnt.*vmcnt\(0\)", i):
                waited = True
                break
            if i.startswith((".LBB", "s_cbranch", "s_branch", "global_", "flat_", "buffer_")):
                break
        assert waited, "the barrier before %r" % code[signal]
    assert barriers[0] < counted < barriers[1]
