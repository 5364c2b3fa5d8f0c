"""Which kernel an SDDMM plan with column slices takes for a call, over all pairs of the feature size the plan was made for
and the one it is called with: the host rule of csrc/sddmm_slice_shape.h, compiled alone."""
import os
import subprocess

import numpy as np
import pytest

from paper_2207_04606_amd import build as sptir_build

HERE = os.path.dirname(os.path.abspath(__file__))
LDS_BYTES = 160 * 1024
GROUP_LANES, QUAD = 8, 4          # lanes of a group, floats of a lane's load


@pytest.fixture(scope="module")
def choices(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("shape") / "shape")
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-I", sptir_build.CSRC, "-o", exe,
                           os.path.join(HERE, "sddmm_slice_shape_main.cpp")])
    out = subprocess.run([exe, "300", "1100"], check=True, capture_output=True, text=True).stdout
    return np.array(out.split(), dtype=np.int64).reshape(-1, 4)


def test_the_lanes_hold_every_feature(choices):
    """A group's lanes hold all floats of a row, and no float4 more than they need, wherever the LDS kernel is chosen."""
    hint, feat, width, lane_quads = choices.T
    in_lds = lane_quads > 0
    assert in_lds.any() and (~in_lds).any()
    assert (lane_quads[in_lds] * GROUP_LANES * QUAD >= feat[in_lds]).all()
    assert ((lane_quads[in_lds] - 1) * GROUP_LANES * QUAD < feat[in_lds]).all()
    assert lane_quads.max() <= 8                          # (the variants that are compiled)
    assert (feat[in_lds] >= QUAD).all()                   # (a row's last float4 is its last four floats)


def test_the_slice_fits_lds(choices):
    hint, feat, width, lane_quads = choices.T
    in_lds = lane_quads > 0
    quads = -(-feat // QUAD)
    stride = np.where(quads % 16 == 0, quads + 8, quads)
    assert (16 * (width * stride + 1)[in_lds] <= LDS_BYTES).all()
    # the size a plan was made for is always taken from LDS
    same = (hint == feat) & (width > 0) & (feat >= QUAD)
    assert in_lds[same].all()
    assert (width[hint > 256] == 0).all() and (width[hint <= 256] >= 1).all()
