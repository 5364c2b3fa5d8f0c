"""The host rules of an SDDMM plan with column slices (csrc/sddmm_slice_shape.h, compiled alone): which kernel takes a call, over
all pairs of the feature size the plan was made for and the one it is called with; where slices are chosen; how the work is
dealt to workgroups."""
import os
import subprocess

import numpy as np
import pytest

from paper_2207_04606_amd import build as sptir_build

HERE = os.path.dirname(os.path.abspath(__file__))
LDS_BYTES = 160 * 1024
GROUP_LANES, QUAD = 8, 4          # lanes of a group, floats of a lane's load


@pytest.fixture(scope="module")
def rules(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("shape") / "shape")
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-I", sptir_build.CSRC, "-o", exe,
                           os.path.join(HERE, "sddmm_slice_shape_main.cpp")])

    def ask(*args, text=None):
        out = subprocess.run([exe, *map(str, args)], check=True, capture_output=True, text=True, input=text).stdout
        return np.array(out.split(), dtype=np.int64)

    return ask


@pytest.fixture(scope="module")
def choices(rules):
    return rules("shape", 300, 1100).reshape(-1, 4)


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


@pytest.mark.parametrize("n_cols,feat,n_long,long_nnz,units,per_segment,slices,half_in,before,after", [
    (9696, 96, 9000, 1_930_000, 900, 5.7, 24, 12, 0, 0),     # Yt of 3.7 MB: lists gather it from L2 (42 us, 66 with slices)
    (7873, 160, 7800, 2_530_000, 900, 5.7, 24, 12, 0, 0),
    (25117, 96, 23000, 13_170_000, 2074, 6.2, 61, 30, 1, 1),  # 9.6 MB
    (25117, 96, 23000, 13_170_000, 2074, 6.2, 61, 15, 1, 0),  # (a hot range)
    (34000, 96, 30000, 14_000_000, 2074, 6.2, 83, 1, 1, 1),  # 13 MB
    (25117, 96, 23000, 13_170_000, 2074, 3.5, 61, 16, 1, 0),  # uneven: half of the segments in less than 42 % of the slices, below 10 MB
    (50642, 48, 23604, 16_520_000, 2108, 5.9, 62, 17, 1, 0),  # (312 us, 663 with slices)
    (27625, 100, 19864, 11_876_000, 2100, 5.3, 70, 10, 1, 1),  # (806 us, 1,645 without)
    (27306, 96, 23000, 13_170_000, 2074, 5.7, 61, 25, 1, 0),  # 10 MB, but for a row
    (27306, 96, 23000, 13_170_000, 2074, 5.7, 50, 21, 1, 1),  # (42 % of the slices)
    (27306, 96, 23000, 13_170_000, 2074, 5.7, 51, 21, 1, 0),
    (27307, 96, 23000, 13_170_000, 2074, 5.7, 61, 25, 1, 1),
    (25117, 96, 23000, 13_170_000, 2074, 3.5, 61, 30, 1, 1),  # short segments: only where a float4 is partly used
    (25000, 100, 23000, 13_170_000, 2074, 3.5, 64, 32, 1, 0),
    (25000, 100, 23000, 13_170_000, 2074, 4.8, 64, 32, 1, 1),
    (34000, 100, 30000, 14_000_000, 2074, 3.5, 86, 43, 1, 1),
    (33007, 128, 1100, 1_050_000, 134, 5.5, 134, 67, 1, 0),    # too few units (86 us, 115 with slices)
    (33007, 128, 1100, 1_050_000, 160, 5.5, 134, 67, 1, 1),
    (232965, 128, 60000, 70_000_000, 3000, 5.9, 940, 470, 1, 1),
    (3001, 128, 531, 1_200_000, 13, 7.9, 13, 1, 1, 1),      # few long rows
    (3001, 128, 531, 1_000_000, 13, 7.9, 13, 1, 0, 0),      # fewer entries than slices need
    (232965, 32, 60000, 70_000_000, 3000, 5.9, 940, 470, 0, 0),  # too few features
    (2**31 - 1, 256, 2**31 - 1, 2**31 - 1, 2**31 - 1, 1.0, 2**31 - 1, 2**31 - 1, 1, 1),
])
def test_where_slices_are_chosen(rules, n_cols, feat, n_long, long_nnz, units, per_segment, slices, half_in, before, after):
    assert rules("pay", n_cols, feat, n_long, long_nnz, units, int(long_nnz / per_segment), slices, half_in).tolist() == [before, after]


@pytest.mark.parametrize("n_slices,parts,hot,most", [(1, 1, 0, 1), (1, 3, 0, 40), (7, 2, 3, 50), (8, 1, 7, 64), (61, 9, 5, 300),
                                                     (61, 9, 60, 1), (200, 3, 0, 10**9), (9, 4, None, 25)])
def test_units_hold_every_segment_once(rules, n_slices, parts, hot, most):
    """No unit has more than `most` segments, each lies in the slice it names, what is not cut stays with the XCD of its
    slice, and none of the 8 XCDs has much more than the others where a slice is hot."""
    rng = np.random.default_rng(n_slices * parts)
    n = rng.integers(0, 30, (parts, n_slices))
    n[rng.random(n.shape) < 0.2] = 0
    if hot is not None:
        n[:, hot] = 1700
    begin = np.concatenate([[0], np.cumsum(n)])
    units = rules("units", n_slices, parts, most, text=" ".join(map(str, begin))).reshape(-1, 3)
    slice_of = np.repeat(np.tile(np.arange(n_slices), parts), n.ravel())
    per_xcd = -(-n_slices // 8)
    by_load = np.sort(n.sum(axis=0))[::-1].cumsum()
    assert rules("half", n_slices, parts, text=" ".join(map(str, begin))) == [1 + int((2 * by_load < n.sum()).sum())]
    seen = np.zeros(begin[-1], dtype=int)
    load = np.zeros(8, dtype=int)
    for i, (s, lo, hi) in enumerate(units):
        assert 0 <= hi - lo <= most
        seen[lo:hi] += 1
        assert (slice_of[lo:hi] == s).all()
        load[i % 8] += hi - lo
        if hi > lo and lo in begin and hi in begin:
            assert i % 8 == s // per_xcd
    assert (seen == 1).all()
    if hot is not None and most < 1000:
        assert load.max() - load.min() <= max(most, n.sum() // 8)


@pytest.mark.parametrize("begin,end,is_long", [(0, 300, 1), (700, 1000, 1), (0, 299, 0), (5, 5, 0), (600, 300, 0),
                                               (-1, 300, 0), (-400, 0, 0), (700, 1001, 0), (1000, 1300, 0),
                                               (-2**31, 2**31 - 1, 0), (2**31 - 1, -2**31, 0)])
def test_rows_outside_the_entries_are_not_long(rules, begin, end, is_long):
    """Row pointers are not validated when a plan is built: a row that is not inside the entries is not searched."""
    assert rules("long", begin, end, 1000, 300) == [is_long]
