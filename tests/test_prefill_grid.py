"""Where the workgroups of the masked attention's kernels come to lie, played through on the host with the kernels' own arithmetic."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_2510_13797_amd", "csrc")


@pytest.fixture(scope="module")
def grids(tmp_path_factory):
    cxx = shutil.which("g++") or shutil.which("c++")
    if cxx is None:
        pytest.skip("no host compiler")
    exe = str(tmp_path_factory.mktemp("grid") / "prefill_grid_model")
    subprocess.check_call([cxx, "-std=c++17", "-O2", "-Wall", "-Werror", "-I", CSRC, "-o", exe, os.path.join(HERE, "prefill_grid_model.cpp")])
    lines = subprocess.check_output([exe], timeout=300).decode().split("\n")
    return [dict((k, int(v)) for k, v in (x.split("=") for x in l.split())) for l in lines if l]


def test_every_row_of_a_grid_has_every_pair_once(grids):
    assert len(grids) > 300 and all(g["once"] for g in grids)


def test_a_pairs_workgroups_come_to_all_shader_engines(grids):
    for g in grids:
        if g["stride"] // 8 % 2:           # an odd number of pairs an XCD: one engine after the other
            assert g["run"] == 4, g
        elif g["stride"] > 16 or g["splits"] > 1:
            assert g["engines"] == 4 and g["most"] <= 340, g
        else:                              # two pairs an XCD, one workgroup of a pair a row
            assert g["engines"] >= 2 and g["most"] <= 500, g
