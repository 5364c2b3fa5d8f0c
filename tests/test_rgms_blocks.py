"""RGMS: rows of Y per block (csrc/rgms_blocks.h, compiled alone).  Whatever their number, a call takes no more passes over X than with the power of
two rows that the rule on entries names, and the rows of Y fit the LDS of a CU as often as theirs."""
import os
import subprocess

import numpy as np
import pytest

from paper_2207_04606_amd import build as sptir_build

HERE = os.path.dirname(os.path.abspath(__file__))
ENTRIES = {5: 1.5, 6: 0.7, 7: 0.35, 8: 0.18, 9: 0.044}  # per relation and row: blocks of 2^5, 2^6, .. rows
D_OUT = np.array([32, 64, 96, 128, 160, 192, 256, 288, 512])
LDS = 160 * 1024


@pytest.fixture(scope="module")
def blocks(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("blocks") / "blocks")
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-Wno-unused-function", "-I", sptir_build.CSRC,
                           "-o", exe, os.path.join(HERE, "rgms_blocks_main.cpp")])

    def ask(rows, *what):  # (n_rows, n_rel, nnz, workspace), or "waves": (kind, ordered, workgroups, tiles_each)
        text = "\n".join(" ".join(str(v) for v in row) for row in rows)
        out = subprocess.run([exe, *what], input=text, check=True, capture_output=True, text=True).stdout
        return np.array(out.split(), dtype=np.int64).reshape(len(rows), -1)

    return ask


def graphs(log2_rows, workspace):
    per_row = ENTRIES[log2_rows] / (2 if workspace else 1)
    most = 500 if log2_rows >= 8 else 1400
    n_rows = np.unique([(b << log2_rows) + d for b in range(162, most) for d in (0, -1, -(1 << log2_rows) // 2)])
    return [(n, 3, int(per_row * 3 * n), int(workspace)) for n in n_rows.tolist()]


@pytest.mark.parametrize("log2_rows,workspace", [(s, w) for s in sorted(ENTRIES) for w in (False, True) if not (s == 9 and w)])
def test_no_more_passes_over_x_than_with_a_power_of_two(blocks, log2_rows, workspace):
    rows, cols, power, cols_of_power = blocks(graphs(log2_rows, workspace)).T
    assert (power == 1 << log2_rows).all()
    assert (cols % 32 == 0).all() and (cols >= 32).all() and (rows >= 1).all() and (rows <= 512).all()
    passes = -(-D_OUT // cols[:, None])
    assert (passes <= -(-D_OUT // cols_of_power[:, None])).all()
    # two workgroups' rows of Y (and the one for places without an entry) in a CU; one's of large blocks, and where there is a block for each
    lds, blocks_of = 8 * cols * (rows + 1), -(-np.array(graphs(log2_rows, workspace))[:, 0] // rows)
    assert (np.where((rows > 256) | (blocks_of <= 256), 1, 2) * lds <= LDS).all()
    assert (2 * rows > power).all() and (4 * rows <= 5 * power).all()
    assert (rows != power).any() != (workspace and log2_rows == 5)  # (those of 32 rows stay as they are with one)


def test_blocks_of_a_whole_turn_have_the_wavefronts_of_those_they_stand_for(blocks):
    """192 to 255 blocks become 256 with as many fewer tiles each."""
    pairs = [(b, t) for b in range(192, 256) for t in range(16, 200)]
    assert (blocks([(0, 0, b, t) for b, t in pairs], "waves") == 16).all()
    assert (blocks([(0, 0, 256, -(-t * b // 256)) for b, t in pairs], "waves") == 16).all()
    for kind, ordered, workgroups, tiles, waves in ((1, 0, 200, 5, 16), (2, 0, 200, 12, 16), (2, 0, 200, 11, 8), (2, 0, 321, 50, 8), (0, 0, 320, 12, 16), (0, 0, 320, 11, 8),
                                                    (0, 1, 320, 16, 16), (0, 1, 320, 15, 8), (0, 0, 321, 12, 8), (0, 0, 1024, 8, 8),
                                                    (0, 0, 1024, 7, 4), (0, 0, 1025, 23, 4), (0, 0, 1025, 24, 8)):
        assert blocks([(kind, ordered, workgroups, tiles)], "waves") == waves
