"""Chunk lists a wavefront per workgroup and four (csrc/list_waves.h), in a single launch over two partitions: both sides of the numbers of
entries, for even and uneven lists that no wavefronts share, with row blocks that are no multiple of four.  Y against the fp64 oracle, the same bit
for bit through every entry point."""
import numpy as np
import pytest
import torch

import oracle
import workloads
from gpu_helpers import assert_y_close, upload
from test_gpu_parity import say

pytestmark = pytest.mark.gpu

N_COLS = 65536  # 8 MB of a feature tile


@pytest.mark.parametrize("n_lists", [4001, 4098])
@pytest.mark.parametrize("even,entries", [(True, 599), (True, 600), (False, 599), (False, 600)])
@pytest.mark.parametrize("feat", [32, 64, 128])
def test_both_sides(gpu_lib, n_lists, even, entries, feat):
    say(f"[list waves] {n_lists} lists of {entries} entries, even={even}, feat={feat}")
    n_rows = 8 * n_lists
    deg = np.full(n_rows, entries // 8)
    deg[::8] += entries - 8 * (entries // 8)
    if not even:  # one list in 64 has three times as many, the others fewer
        deg[:] = entries // 8 - 1
        deg[0::512] *= 16
    w = workloads.random_csr(n_rows, N_COLS, deg, n_lists, feat)
    d = upload(w)
    Yr, Sr = oracle.spmm_csr(w.n_rows, w.indptr, w.indices, w.values, w.X)
    hyb = gpu_lib.sptir_hyb_build_ex(n_rows, N_COLS, d.indptr, d.indices, d.values, 2, 4,
                                     dict(row_block=8, rounds=2, parts_per_launch=2, heavy_len=2048, column_slices=2))
    info = gpu_lib.sptir_hyb_info(hyb)
    assert info["n_phases"] == 1 and info["rounds"] == 0 and info["n_row_blocks"] == n_lists
    Y = torch.full((n_rows, feat), float("nan"), device="cuda")
    gpu_lib.sptir_spmm(hyb, d.X, Y)
    assert_y_close(Y.cpu().numpy(), Yr, Sr, what=f"{n_lists} lists")
    again = torch.full_like(Y, float("nan"))
    list_waves = gpu_lib.sptir_spmm_timed(hyb, d.X, again)["list_waves"]
    assert list_waves == 1 or (feat == 32 and not even)  # (a list for several wavefronts would be another kernel)
    assert torch.equal(Y, again)
    again.fill_(float("nan"))
    gpu_lib.sptir_spmm_noalloc(hyb, d.X, again)
    assert torch.equal(Y, again)
    hyb.destroy()
