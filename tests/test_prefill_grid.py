"""Where the workgroups of the masked attention's kernels come to lie, played through on the host with the kernels' own arithmetic."""
import os
import shutil
import subprocess

import numpy as np
import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_2510_13797_amd", "csrc")


@pytest.fixture(scope="module")
def model(tmp_path_factory):
    cxx = shutil.which("g++") or shutil.which("c++")
    if cxx is None:
        pytest.skip("no host compiler")
    exe = str(tmp_path_factory.mktemp("grid") / "prefill_grid_model")
    subprocess.check_call([cxx, "-std=c++17", "-O2", "-Wall", "-Werror", "-I", CSRC, "-o", exe, os.path.join(HERE, "prefill_grid_model.cpp")])

    def run(*args, lines=()):
        text = "".join(" ".join(str(int(x)) for x in l) + "\n" for l in lines)
        out = subprocess.run([exe, *args], input=text.encode(), stdout=subprocess.PIPE, timeout=300, check=True).stdout.decode()
        return [dict((k, int(v)) for k, v in (x.split("=") for x in l.split())) for l in out.split("\n") if l]
    return run


@pytest.fixture(scope="module")
def grids(model):
    return model("pairs")


def test_every_row_of_a_grid_has_every_pair_once(grids):
    assert len(grids) > 300 and all(g["once"] for g in grids)


def test_a_pairs_workgroups_come_to_all_shader_engines(grids):
    for g in grids:
        if g["stride"] // 8 % 2:           # an odd number of pairs an XCD: one engine after the other
            assert g["run"] == 4, g
        else:
            assert g["engines"] == 4 and g["most"] <= 340 and (g["run"] == 4 or (g["stride"], g["splits"]) != (16, 1)), g


def in_one_launch(B, Hq, Hkv, total_rows):
    """Whether the gradients' two kinds of workgroup are one launch: the GPU tests say with it which side a case is on."""
    g = Hq // Hkv
    heads = 4 if g % 4 == 0 or g == 7 else 2 if g % 2 == 0 else 1
    rows = 32 * (4 // heads) * B
    return -(-total_rows // rows) * B * Hkv * -(-g // heads) <= (512 if B * Hkv <= 4 else 256)


def test_the_side_of_the_line_that_the_gpu_tests_reckon_with(model):
    r = np.random.default_rng(3)
    cases = [(B, g * Hkv, Hkv, int(n)) for B in (1, 2, 4, 5, 16, 67, 130) for g in range(1, 9) for Hkv in (1, 2, 3, 8)
             for n in [*r.integers(B, 700 * B, 20), 32 * B * 32, 32 * B * 32 + 1]]
    got = [bool(x["one"]) for x in model(lines=[(B, Hq, Hkv, 64, n, n, n, 10, 4) for B, Hq, Hkv, n in cases])]
    assert got == [in_one_launch(*c) for c in cases] and 500 < sum(got) < len(got) - 500
    # the batches of the GPU test that lie on the line and one row beyond it
    assert in_one_launch(4, 12, 2, 4 * 640) and not in_one_launch(4, 12, 2, 4 * 640 + 1)
    assert in_one_launch(4, 8, 1, 4 * 2048) and not in_one_launch(4, 8, 1, 4 * 2048 + 1)


def _trajectories(B, Hq, Hkv, d, rows, P, c):
    return [(B, Hq, Hkv, d, sum(rows), max(rows), r, p, x) for r, p, x in zip(rows, P, c)]


def test_parts_of_a_dense_key_block_fit_the_workspace_and_the_grid(model):
    r = np.random.default_rng(20251013)
    lines = []
    for _ in range(4000):
        g, Hkv, B = (int(x) for x in (r.integers(1, 9), r.choice([1, 2, 3, 8]), np.exp(r.uniform(0, np.log(130)))))
        rows = np.exp(r.uniform(0, np.log(r.choice([60, 600, 9000])), B)).astype(np.int64)
        lines += _trajectories(B, g * Hkv, Hkv, r.choice([64, 128]), rows, r.integers(0, 400, B), r.choice([0, 1, 2, 16, 32, 5000], B))
    lines = [lines[i] for i in r.permutation(len(lines))[:60000]]
    got = model(lines=lines)
    assert len(got) == len(lines) and max(x["parts"] for x in got) == 16
    for l, x in zip(lines, got):
        assert 1 <= x["band"] <= x["splits"] and x["sums"] <= x["room"] and x["groups"] <= x["grid"], (l, x)


def test_dense_key_blocks_have_more_than_eight_parts_only_where_each_saves_more_than_its_sums_cost(model):
    # (with parts of eight tiles and up the first three were 5 to 9 % slower than with eight parts; the last is a third faster with sixteen)
    for t in (_trajectories(10, 4, 1, 64, [450, 1153] * 5, [293] * 10, [32] * 10), _trajectories(1, 24, 8, 128, [1229], [110], [16]),
              _trajectories(13, 16, 2, 128, [224, 551] * 6 + [400], [258] * 13, [16] * 13)):
        assert max(x["parts"] for x in model(lines=t)) <= 12
    assert [x["parts"] for x in model(lines=_trajectories(2, 7, 1, 64, [3745, 3961], [100, 100], [32, 32]))] == [16, 16]
    r = np.random.default_rng(5)
    got = model(lines=[_trajectories(*a, r.choice([64, 128]), [n] * a[0], [60] * a[0], [16] * a[0])[0]
                       for a in [(1, 4, 1), (3, 12, 2), (6, 5, 1), (10, 4, 1), (2, 32, 8)] for n in r.integers(100, 6000, 200)])
    more = [x for x in got if x["parts"] > 8]
    assert len(more) > 100
    for x in more:
        assert x["parts"] * 8 <= x["tiles"] and x["parts"] ** 2 * x["bytes"] <= 0.5e6 * x["tiles"] * 1.0001, x
    # groups whose response blocks are whole: no part is shorter than one of those, three tiles a head
    for g in (2, 3, 4, 5):
        assert all(x["parts"] <= 8 or x["parts"] * 3 * g <= x["tiles"]
                   for n in range(200, 3000, 40) for x in model(lines=_trajectories(1, g, 1, 64, [n], [40], [16])))
