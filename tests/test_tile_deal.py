"""How units and feature tiles are dealt to workgroups and XCDs (csrc/tile_deal.h, compiled alone): every unit of every tile once,
whatever the counts; which tile gives units away, and to which XCDs; that an XCD's heavy lists are consecutive."""
import os
import subprocess

import numpy as np
import pytest

from paper_2207_04606_amd import build as sptir_build

HERE = os.path.dirname(os.path.abspath(__file__))
BEYOND_L2 = 1 << 16  # rows of X: 8 MB of a tile


@pytest.fixture(scope="module")
def deal(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("deal") / "deal")
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-Wno-unused-function", "-I", sptir_build.CSRC,
                           "-o", exe, os.path.join(HERE, "tile_deal_main.cpp")])

    def ask(kind, n_units, n_tiles, x=0, feat=128, n_cols=BEYOND_L2):
        args = [exe, "deal", kind, n_units, n_tiles, x, feat, n_cols]
        out = subprocess.run([str(a) for a in args], check=True, capture_output=True, text=True).stdout
        rows = np.array(out.split(), dtype=np.int64).reshape(-1, 3)
        return rows[:-1], rows[-1]

    return ask


UNITS = [1, 2, 7, 8, 9, 63, 64, 65, 511, 512, 513, 514, 515, 516, 517, 518, 519, 520, 2646, 2647, 4099]


def assert_each_once(rows, n_units, n_tiles):
    keys = rows[:, 2] * n_units + rows[:, 1]
    assert (rows[:, 1] >= 0).all() and (0 <= rows[:, 2]).all() and (rows[:, 2] < n_tiles).all()
    assert np.array_equal(np.sort(keys), np.arange(n_units * n_tiles))


@pytest.mark.parametrize("kind", ["plain", "lists", "heavy"])
@pytest.mark.parametrize("n_tiles", [1, 2, 3, 4, 5, 6, 8, 12, 16])
def test_every_unit_of_every_tile_once(deal, kind, n_tiles):
    for n_units in UNITS:
        rows, (grid, moved, _) = deal(kind, n_units, n_tiles, feat=32 * n_tiles)
        assert_each_once(rows, n_units, n_tiles)
        assert (moved > 0) == (kind == "lists" and n_tiles == 4 and n_units >= 512)


@pytest.mark.parametrize("line", range(4))
def test_units_of_the_last_line_go_to_the_other_tiles_xcds(deal, line):
    for n_units in (512, 515, 2647):
        rows, (grid, moved, slow) = deal("lists", n_units, 4, x=4096 + 128 * line)
        assert moved == n_units // 8 and (line + slow) % 4 == 3
        assert_each_once(rows, n_units, 4)
        bid, unit, tile = rows.T
        own = bid % 4 == tile                      # (eight XCDs, two for each of the four tiles)
        assert (own == ((tile != slow) | (unit < n_units - moved))).all()
        helped = np.bincount(bid[~own] % 8, minlength=8)
        helpers = [x for x in range(8) if x % 4 != slow]
        assert helped[[x for x in range(8) if x % 4 == slow]].sum() == 0 and np.ptp(helped[helpers]) <= 1
        for x in helpers:                          # after all units of its own
            mine = bid % 8 == x
            assert bid[mine & own].max() < bid[mine & ~own].min()


@pytest.mark.parametrize("change", [dict(x=4096 + 64), dict(feat=64), dict(feat=160), dict(n_cols=BEYOND_L2 - 1)])
def test_nothing_moves_otherwise(deal, change):
    rows, (_, moved, _) = deal("lists", 1000, 4, **change)
    plain, _ = deal("plain", 1000, 4)
    assert moved == 0 and np.array_equal(rows, plain)


@pytest.mark.parametrize("n_tiles", [2, 4])
def test_the_heavy_lists_of_an_xcd_are_consecutive(deal, n_tiles):
    for n_units in UNITS:
        rows, _ = deal("heavy", n_units, n_tiles)
        for x in range(8):
            units = rows[rows[:, 0] % 8 == x, 1]
            assert np.array_equal(units, np.arange(len(units)) + (units[0] if len(units) else 0))
            assert abs(len(units) - n_units * n_tiles / 8) < 1


def test_a_single_tile_keeps_turns(deal):
    rows, _ = deal("heavy", 100, 1)
    plain, _ = deal("plain", 100, 1)
    assert np.array_equal(rows, plain)
