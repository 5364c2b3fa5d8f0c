"""SpMM where units of the slow line's tile go to other XCDs (csrc/tile_deal.h): below, at and above the number of units from which they
do, a list each, with and without heavy lists, which make more of them move.  Y against the fp64 oracle, bit for bit the same wherever X begins."""
import numpy as np
import pytest
import torch

import oracle
import workloads
from gpu_helpers import assert_y_close, upload
from test_gpu_parity import say

pytestmark = pytest.mark.gpu

N_COLS = 65536  # 8 MB of a feature tile


@pytest.mark.parametrize("heavy", [False, True])
@pytest.mark.parametrize("parts", [1, 2])
@pytest.mark.parametrize("n_rows", [8 * 511, 8 * 512 - 3, 8 * 519 + 5])
def test_units_beside_the_fewest_that_move(gpu_lib, n_rows, parts, heavy):
    say(f"[moved units] {n_rows} rows, {parts} partitions, heavy={heavy}")
    deg = np.full(n_rows, 26)  # 208 entries a list, from 200 on they move
    if heavy:
        deg[np.random.default_rng(n_rows).permutation(n_rows)[:100]] = 2200
    w = workloads.random_csr(n_rows, N_COLS, deg, n_rows, 128)
    d = upload(w)
    Yr, Sr = oracle.spmm_csr(w.n_rows, w.indptr, w.indices, w.values, w.X)
    hyb = gpu_lib.sptir_hyb_build_ex(n_rows, N_COLS, d.indptr, d.indices, d.values, parts, 5,
                                     dict(row_block=8, rounds=2, parts_per_launch=parts, heavy_len=64, column_slices=2))
    info = gpu_lib.sptir_hyb_info(hyb)
    assert info["n_phases"] == 1 and (info["n_heavy_lists"] > 0) == heavy and info["n_row_blocks"] == -(-n_rows // 8)
    first = None
    for line in (0, 32, 64, 96):
        room = torch.empty(d.X.numel() + 128, device="cuda")
        X = room[line:line + d.X.numel()].view_as(d.X)
        X.copy_(d.X)
        Y = torch.full((n_rows, 128), float("nan"), device="cuda")
        gpu_lib.sptir_spmm(hyb, X, Y)
        if first is None:
            assert_y_close(Y.cpu().numpy(), Yr, Sr, what=f"{n_rows} rows")
            first = Y
            again = torch.full_like(Y, float("nan"))
            assert gpu_lib.sptir_spmm_timed(hyb, X, again)["list_waves"] == 1  # (a list for several wavefronts would be another kernel)
            assert torch.equal(Y, again)
        assert torch.equal(Y, first), line
    hyb.destroy()
