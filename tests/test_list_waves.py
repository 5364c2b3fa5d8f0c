"""Wavefronts per workgroup of chunk lists (csrc/list_waves.h, compiled alone): both sides of every number that the rule asks for."""
import os
import subprocess

import pytest

from paper_2207_04606_amd import build as sptir_build

HERE = os.path.dirname(os.path.abspath(__file__))
FIELDS = ("rounds", "n_launches", "parts", "n_cols", "n_lists", "entries", "chunks", "longest", "feat", "tile_floats", "n_tiles")
# 1000 lists of 600 entries, 10 chunks each, over two partitions of an X whose feature tiles of 32 floats have 8 MB
EVEN = dict(rounds=0, n_launches=1, parts=2, n_cols=65536, n_lists=1000, entries=600000, chunks=10000, longest=20, feat=64, tile_floats=32, n_tiles=2)
HALF_ROWS = dict(EVEN, n_cols=32768, entries=300000, chunks=5000, longest=10, feat=100, tile_floats=64)
UNEVEN = dict(EVEN, entries=1280000, chunks=20000, longest=41)


@pytest.fixture(scope="module")
def waves(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("waves") / "waves")
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-Wno-unused-function", "-I", sptir_build.CSRC,
                           "-o", exe, os.path.join(HERE, "list_waves_main.cpp")])

    def ask(lists, **change):
        row = dict(lists, **change)
        out = subprocess.run([exe], input=" ".join(str(row[f]) for f in FIELDS), check=True, capture_output=True, text=True).stdout
        return int(out)

    return ask


@pytest.mark.parametrize("lists", [EVEN, HALF_ROWS, UNEVEN])
def test_one_without_any_of_what_four_need(waves, lists):
    assert waves(lists) == 4
    for change in (dict(n_launches=2), dict(parts=1), dict(n_tiles=1), dict(n_cols=lists["n_cols"] - 1), dict(entries=lists["entries"] - 1)):
        assert waves(lists, **change) == 1, change
        assert waves(lists, rounds=1, **change) == 4, change


def test_lists_that_are_not_even_are_longer(waves):
    assert waves(EVEN, longest=21) == 1 and waves(EVEN, longest=21, entries=1279999) == 1 and waves(EVEN, longest=21, entries=1280000) == 4


@pytest.mark.parametrize("feat,tile_floats,n_tiles,n_cols", [(128, 64, 2, 32768), (20, 16, 2, 131072), (65, 64, 2, 32768), (256, 128, 2, 16384)])
def test_bytes_are_those_of_the_feature_tile(waves, feat, tile_floats, n_tiles, n_cols):
    shape = dict(feat=feat, tile_floats=tile_floats, n_tiles=n_tiles)
    assert waves(EVEN, n_cols=n_cols, **shape) == 4 and waves(EVEN, n_cols=n_cols - 1, **shape) == 1


def test_numbers_of_a_large_graph(waves):
    """2^31 entries in 2^28 lists."""
    large = dict(EVEN, n_lists=1 << 28, entries=(1 << 31) - 1, chunks=1 << 30, longest=1 << 24, n_cols=(1 << 31) - 1)
    assert waves(large) == 1 and waves(dict(large, n_lists=1 << 20)) == 4
