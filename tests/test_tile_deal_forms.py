"""The forms of decode_deal() that the kernels of chunk lists and of heavy lists are built with (csrc/tile_deal.h, compiled alone) name the unit and
the tile that the general form names, which test_tile_deal.py looks at; also with as many units as 32 bits can number."""
import os
import subprocess

import pytest

from paper_2207_04606_amd import build as sptir_build

HERE = os.path.dirname(os.path.abspath(__file__))
UNITS = [1, 2, 3, 7, 8, 9, 64, 65, 511, 512, 513, 519, 2646, 2647, 4099, 1 << 26, (1 << 27) - 1]


@pytest.fixture(scope="module")
def forms(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("forms") / "forms")
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-Wno-unused-function", "-I", sptir_build.CSRC,
                           "-o", exe, os.path.join(HERE, "tile_deal_forms_main.cpp")])
    return exe


@pytest.mark.parametrize("kind", ["plain", "lists", "heavy"])
@pytest.mark.parametrize("n_tiles", [1, 2, 3, 4, 5, 6, 8, 12, 16])
def test_the_forms_agree(forms, kind, n_tiles):
    for n_units in UNITS:
        if n_units * n_tiles > 0x7FFFFFFF:
            continue
        out = subprocess.run([forms, kind, str(n_units), str(n_tiles)], capture_output=True, text=True)
        assert out.returncode == 0 and int(out.stdout) > 0, (n_units, out.returncode)
