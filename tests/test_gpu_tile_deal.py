"""SpMM where the last line of every 512 bytes of X has its units dealt to the XCDs of the other tiles, and heavy lists go to the XCDs
by ranges (csrc/tile_deal.h): at the number of units from which they move and beside it, for every line that X can begin at.  Y against
the fp64 oracle, and bit for bit the same for every beginning."""
import numpy as np
import pytest
import torch

import oracle
import workloads
from gpu_helpers import assert_y_close, upload
from test_gpu_parity import say

pytestmark = pytest.mark.gpu

N_COLS = 65536  # 8 MB of a feature tile, from where on units move


@pytest.mark.parametrize("rounds", [1, 2])
@pytest.mark.parametrize("n_rows", [8 * 4 * 511, 8 * 4 * 512 - 31, 8 * 4 * 519 + 5])
def test_units_that_move(gpu_lib, n_rows, rounds):
    say(f"[tile deal] {n_rows} rows, rounds option {rounds}")
    rng = np.random.default_rng(n_rows)
    deg = rng.integers(0, 6, n_rows)
    deg[rng.permutation(n_rows)[:300]] = rng.integers(65, 300, 300)
    w = workloads.random_csr(n_rows, N_COLS, deg, n_rows, 128)
    d = upload(w)
    Yr, Sr = oracle.spmm_csr(w.n_rows, w.indptr, w.indices, w.values, w.X)
    hyb = gpu_lib.sptir_hyb_build_ex(n_rows, N_COLS, d.indptr, d.indices, d.values, 2, 6,
                                     dict(row_block=8, rounds=rounds, parts_per_launch=2, heavy_len=20, column_slices=2))
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
        assert torch.equal(Y, first), line
    hyb.destroy()
