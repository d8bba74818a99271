"""The module _native is a faster way into the library, not a condition for it: without one, or with one made for
another torch, the package loads, says so, and calls through ctypes."""
import os
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def imported(before):
    code = before + """
import warnings
with warnings.catch_warnings(record=True) as seen:
    warnings.simplefilter("always")
    from paper_2504_06443_amd import binding
parts, waves = binding.spmm_partition_counts([400, 4, 4], 3, 1000, 1)
print(sum("_native" in str(w.message) for w in seen), binding._native.__name__, waves)
"""
    run = subprocess.run([sys.executable, "-c", code], cwd=ROOT, capture_output=True, text=True, timeout=300)
    assert run.returncode == 0, run.stderr
    return run.stdout.split()


@pytest.mark.parametrize("before", [
    "import sys; sys.modules['paper_2504_06443_amd._native'] = None",              # does not load
    "import paper_2504_06443_amd.build as build; build.NATIVE += '.none'",             # is not there
    "import paper_2504_06443_amd.build as build; build.built_for = lambda: '_native for torch 0'"])
def test_the_package_loads_without_it(before):
    assert imported(before) == ["1", "_ThroughCtypes", "1"]


def test_a_module_of_another_torch_is_not_current(tmp_path, monkeypatch):
    import paper_2504_06443_amd.build as build
    monkeypatch.setattr(build, "NATIVE", str(tmp_path / "_native.so"))
    made = []
    monkeypatch.setattr(build, "build_native", lambda: made.append(1))
    for content in (None, b"_native for torch 1.0, Python 3.10\0", build.built_for().encode() + b"0\0"):
        if content is not None:
            (tmp_path / "_native.so").write_bytes(b"\x7fELF" + content)
        build.build_missing()
    assert len(made) == 3
    (tmp_path / "_native.so").write_bytes(b"\x7fELF" + build.built_for().encode() + b"\0")
    build.build_missing()
    assert len(made) == 3


def test_the_built_one_serves():
    assert imported("") == ["0", "paper_2504_06443_amd._native", "1"]
