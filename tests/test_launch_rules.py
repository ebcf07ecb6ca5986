"""Workgroup sizes of the persistent kernels (host rules, no GPU): a cap on the
workgroups keeps meaning workgroups of four waves unless the caller says eight,
and an explicit size is what is launched."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def waves(tmp_path_factory):
    if shutil.which("g++") is None:
        pytest.skip("g++ not available")
    exe = tmp_path_factory.mktemp("rules") / "launch_rules"
    subprocess.run(["g++", "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
                    "-I", os.path.join(ROOT, "paper_1209_3314_amd", "csrc"),
                    os.path.join(ROOT, "tests", "launch_rules.cpp"), "-o", str(exe), "-L/opt/rocm/lib", "-lamdhip64",
                    "-Wl,-rpath,/opt/rocm/lib"], check=True)

    def run(wg_waves, blocks, tiles, cus=256):
        out = subprocess.run([str(exe)] + [str(v) for v in (wg_waves, blocks, tiles, cus)], check=True, capture_output=True,
                             text=True)
        return tuple(int(v) for v in out.stdout.split())

    return run


@pytest.mark.parametrize("tiles", [1, 512, 513, 100000])
def test_waves(waves, tiles):
    for blocks in (0, 1, 512, 100000):
        assert waves(4, blocks, tiles) == (4, 4) and waves(8, blocks, tiles) == (8, 8)
    for blocks in (1, 512, 100000):
        assert waves(0, blocks, tiles) == (4, 4)
    assert waves(0, 0, tiles)[0] == 8


def test_automatic_edt_size_by_tiles(waves):
    """Eight waves as long as every tile's workgroup is resident: two a compute unit."""
    for cus in (32, 64, 256):
        assert waves(0, 0, 1, cus)[1] == 8 and waves(0, 0, 2 * cus, cus)[1] == 8
        assert waves(0, 0, 2 * cus + 1, cus)[1] == 4 and waves(0, 0, 100000, cus)[1] == 4


def test_tuner_candidates_differ():
    from paper_1209_3314_amd import tune

    for cands in tune.GRID.values():
        keys = [tuple(sorted(dict(tune.DEFAULTS, **c).items())) for c in cands]
        assert len(set(keys)) == len(keys)
        # the automatic size under a cap is four waves: not a candidate beside four waves
        assert not any(c.get("persistent_blocks") and c["wg_waves"] == 0 for c in cands)
