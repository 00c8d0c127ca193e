"""How the workgroups of a decode step agree that a sequence is done, played through on the host.

The kernels' arithmetic (which rows are a workgroup's, who counts where, how many are waited for) is compiled
for the host and every order in which the waves of a sequence can read its tables and count is followed: no
order may move the tables twice or not at all, fold a partial result that is not written, or leave a counter
that is not zero.
"""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_2510_13797_amd", "csrc")


@pytest.fixture(scope="module")
def model(tmp_path_factory):
    cxx = shutil.which("g++") or shutil.which("c++")
    if cxx is None:
        pytest.skip("no host compiler")
    exe = str(tmp_path_factory.mktemp("model") / "decode_count_model")
    subprocess.check_call([cxx, "-std=c++17", "-O2", "-Wall", "-Werror", "-I", CSRC, "-o", exe,
                           os.path.join(HERE, "decode_count_model.cpp")])

    def run(*args):
        lines = subprocess.check_output([exe, *args], timeout=300).decode().split("\n")
        return [dict((k, int(v)) for k, v in (x.split("=") for x in l.split())) for l in lines if l]
    return run


def test_no_order_of_a_sequences_workgroups_leaves_a_counter_or_moves_the_tables_early(model):
    rows = model()
    assert len(rows) > 200 and max(r["states"] for r in rows) > 1000
    assert [r for r in rows if r["bad"]] == []


def test_the_model_shows_workgroups_without_rows_that_are_not_counted(model):
    # the mistake it is there for: cut plans whose sequences come to a cut line in the step
    rows = model("uncounted")
    bad = [r for r in rows if r["bad"]]
    assert bad and all(r["chunks"] > 1 for r in bad)
    assert any(r["L"] == 31 and r["waves"] == 1 for r in bad)      # 32 rows whole, 33 in two chunks
