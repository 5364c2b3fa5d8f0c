"""Workgroups of one wavefront and of four for chunk lists in a single launch over two partitions: on both sides of the number of entries
from which its lists are taken four at a time, and with row blocks that are no multiple of four.  Y against the fp64 oracle, the same bit
for bit through every entry point."""
import numpy as np
import pytest
import torch

import oracle
import workloads
from gpu_helpers import assert_y_close, upload
from test_gpu_parity import say

pytestmark = pytest.mark.gpu

N_COLS = 65536      # 8 MB of a feature tile, from where on lists may be in step
LIST_ENTRIES = 1280  # and so many entries a list


@pytest.mark.parametrize("n_lists", [1, 3, 5, 34])
@pytest.mark.parametrize("entries", [LIST_ENTRIES - 1, LIST_ENTRIES])
@pytest.mark.parametrize("feat", [41, 128])
def test_both_sides(gpu_lib, n_lists, entries, feat):
    say(f"[in step] {n_lists} lists of {entries} entries, feat={feat}")
    n_rows = 8 * n_lists
    rng = np.random.default_rng(n_lists + entries)
    deg = rng.multinomial(entries * n_lists, np.full(n_rows, 1 / n_rows))
    w = workloads.random_csr(n_rows, N_COLS, deg, n_lists, feat)
    d = upload(w)
    Yr, Sr = oracle.spmm_csr(w.n_rows, w.indptr, w.indices, w.values, w.X)
    hyb = gpu_lib.sptir_hyb_build_ex(n_rows, N_COLS, d.indptr, d.indices, d.values, 2, 4,
                                     dict(row_block=8, rounds=2, parts_per_launch=2, heavy_len=2048, column_slices=2))
    Y = torch.full((n_rows, feat), float("nan"), device="cuda")
    gpu_lib.sptir_spmm(hyb, d.X, Y)
    assert_y_close(Y.cpu().numpy(), Yr, Sr, what=f"{n_lists} lists")
    for other in (gpu_lib.sptir_spmm_timed, gpu_lib.sptir_spmm_noalloc):
        again = torch.full_like(Y, float("nan"))
        other(hyb, d.X, again)
        assert torch.equal(Y, again)
    hyb.destroy()
