"""Heavy lists that share a launch with the last of the chunk lists: more of them than chunk lists and fewer, in one launch, in rounds,
after other launches, and where one sweep over the features is not enough.  Y against the fp64 oracle, and bit for bit against the
timed call, which launches each kind by itself."""
import numpy as np
import pytest
import torch

import oracle
import workloads
from gpu_helpers import upload
from test_gpu_parity import assert_y_close, say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("options", [{"rounds": 2}, {"rounds": 1}, {"rounds": 2, "parts_per_launch": 1},
                                     {"rounds": 1, "wide_stream": 1}, {"rounds": 2, "row_block": 8}])
@pytest.mark.parametrize("feat", [1, 4, 17, 41, 128, 131, 600])
@pytest.mark.parametrize("n_rows,n_heavy", [(1, 1), (33, 33), (700, 9), (700, 400), (4100, 2600)])
def test_heavy_with_lists(gpu_lib, n_rows, n_heavy, feat, options):
    say(f"[heavy with lists] {n_rows} rows, {n_heavy} heavy, feat={feat} {options}")
    rng = np.random.default_rng(n_rows + feat)
    deg = rng.integers(0, 9, n_rows)
    deg[rng.permutation(n_rows)[:n_heavy]] = rng.integers(65, 400, n_heavy)
    w = workloads.random_csr(n_rows, 2100, deg, feat, feat)
    d = upload(w)
    Yr, Sr = oracle.spmm_csr(w.n_rows, w.indptr, w.indices, w.values, w.X)
    hyb = gpu_lib.sptir_hyb_build_ex(n_rows, 2100, d.indptr, d.indices, d.values, 3, 11,
                                     dict(options, heavy_len=20, column_slices=2))
    assert gpu_lib.sptir_hyb_info(hyb)["n_heavy_pieces"] >= n_heavy
    Y = torch.full((n_rows, feat), float("nan"), device="cuda")
    gpu_lib.sptir_spmm(hyb, d.X, Y)
    assert_y_close(Y.cpu().numpy(), Yr, Sr, what=f"{options} feat={feat}")
    for other in (lambda y: gpu_lib.sptir_spmm_timed(hyb, d.X, y), lambda y: gpu_lib.sptir_spmm_noalloc(hyb, d.X, y)):
        again = torch.full_like(Y, float("nan"))
        other(again)
        assert torch.equal(Y, again)
    hyb.destroy()
