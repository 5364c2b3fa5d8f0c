"""How many units of the slow line's tile go to the XCDs of the others (csrc/tile_deal.h, compiled alone): an eighth (a single partition: a
sixteenth), more where heavy lists have more entries than the others, up to a quarter; none of short lists; and every unit is dealt once."""
import os
import subprocess

import pytest

from paper_2207_04606_amd import build as sptir_build

HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.fixture(scope="module")
def moved(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("share") / "share")
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-Wno-unused-function", "-I", sptir_build.CSRC,
                           "-o", exe, os.path.join(HERE, "tile_deal_share_main.cpp")])
    return lambda *args: int(subprocess.run([exe, *map(str, args)], check=True, capture_output=True, text=True).stdout)


@pytest.mark.parametrize("n_units", [512, 515, 2646, 4099])
def test_share(moved, n_units):
    entries = 200 * n_units
    for heavy, one, several in ((0, 1, 2), (entries // 2, 1.5, 2), (entries, 2, 2), (2 * entries, 3, 3), (3 * entries, 4, 4), (9 * entries, 4, 4)):
        assert moved(n_units, entries, heavy, n_units, 1) == int(n_units * one / 16)
        assert moved(n_units, entries, heavy, n_units, 0) == int(n_units * several / 16)


def test_none_of_short_lists(moved):
    assert moved(2646, 200 * 2646 - 1, 0, 2646, 0) == 0 and moved(2646, 0, 1000, 0, 0) == 0 and moved(511, 200 * 511, 0, 511, 0) == 0
    assert moved(660, 200 * 2640, 0, 2640, 0) == 82 and moved(660, 200 * 2640 - 1, 0, 2640, 0) == 0  # (four lists a unit)
    assert moved(2646, (1 << 31) - 1, (1 << 31) - 1, 2646, 1) == 330
