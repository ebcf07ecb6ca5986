"""The grid barrier's protocol (csrc/iwpp_barrier.hpp), run on the CPU with the
workgroups' memory operations in random order: a workgroup leaves a barrier with
exactly the list lengths appended before it, however long it was held up while
others went on.  A protocol with one word per group, which a group that is a
barrier ahead writes over, fails in the same model."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_late_pollers_see_their_own_generation(tmp_path):
    if shutil.which("g++") is None:
        pytest.skip("g++ not available")
    exe = tmp_path / "barrier_model"
    subprocess.run(["g++", "-std=c++17", "-O2", "-Wall", "-I", os.path.join(ROOT, "paper_1209_3314_amd", "csrc"),
                    os.path.join(ROOT, "tests", "barrier_model.cpp"), "-o", str(exe)], check=True)
    out = subprocess.run([str(exe)], check=True, capture_output=True, text=True, timeout=100).stdout
    got = dict(l.split() for l in out.splitlines())
    assert int(got["library"]) == 0, out
    assert int(got["one_word"]) > 0, out  # the model does hold workgroups up long enough
