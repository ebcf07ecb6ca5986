"""Scratch of a distance transform (host rules, no GPU): no image needs more than
26 x 26 tiles with 344 bytes of lists, stamps and change records each would take
-- what a server's scratch area was sized for stays admitted -- and what a launch
lays out fits what admission counts."""
import os
import random
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def limits(h, w):
    """(admission, launch) bytes with 26 x 26 tiles."""
    t = -(-h // 26) * -(-w // 26)
    a256 = lambda n: -(-n // 256) * 256
    return 344 * t + 20 * 256 + 8 * h * w + 2 * 256 + 56, a256(2 * (a256(4 * h * w) + 256) + 21 * a256(4 * t) + 256 * t)


def sizes():
    r = random.Random(5)
    edges = [1, 2, 16, 17, 26, 27, 32, 33, 47, 48, 49, 50, 52, 53, 64, 65, 80, 81, 96, 97, 104, 105, 145, 389]
    out = [(h, w) for h in edges for w in edges]
    for n in edges:
        out += [(n, 40000), (40000, n), (n, 4096), (4096, n)]
    out += [(r.randint(1, 300), r.randint(1, 300)) for _ in range(800)]
    out += [(r.randint(1, 20000), r.randint(1, 20000)) for _ in range(300)]
    return out + [(4096, 4096), (30000, 30000), (46340, 1), (1, 46340)]


def test_no_size_needs_more_than_before(tmp_path):
    if shutil.which("g++") is None:
        pytest.skip("g++ not available")
    from paper_1209_3314_amd import _lib

    if not os.path.exists(_lib.LIB_PATH):
        from paper_1209_3314_amd import build

        build.build()
    pkg = os.path.dirname(_lib.LIB_PATH)
    exe = tmp_path / "scratch_rules"
    subprocess.run(["g++", "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", "-I", os.path.join(pkg, "csrc"),
                    os.path.join(ROOT, "tests", "scratch_rules.cpp"), "-o", str(exe), _lib.LIB_PATH,
                    "-L/opt/rocm/lib", "-lamdhip64", f"-Wl,-rpath,{pkg}:/opt/rocm/lib"], check=True)
    todo = sizes()
    out = subprocess.run([str(exe)] + [str(v) for s in todo for v in s], check=True, capture_output=True, text=True).stdout
    got = [tuple(int(v) for v in l.split()) for l in out.splitlines()]
    assert [g[:2] for g in got] == todo
    for h, w, admitted, laid_out in got:
        was_admitted, was_laid_out = limits(h, w)
        assert admitted <= was_admitted, (h, w, admitted, was_admitted)
        assert laid_out <= was_laid_out, (h, w, laid_out, was_laid_out)
        assert laid_out <= admitted + 64 * 256, (h, w)
