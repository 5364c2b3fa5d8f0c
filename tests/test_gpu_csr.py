"""SpMM straight from CSR against the fp64 oracle at the edges of its row classes and feature tiles."""
import numpy as np
import pytest
import torch

import oracle
import workloads
from gpu_helpers import assert_y_close, upload

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_rows", [1, 63, 65, 200])
@pytest.mark.parametrize("n_cols,feat", [(3000, 1), (3000, 3), (3000, 4), (3000, 16), (3000, 17), (3000, 35), (3000, 160),
                                         (60_000, 36), (60_000, 41), (60_000, 67)])
def test_row_lengths_and_tails(gpu_lib, n_rows, n_cols, feat):
    """Lengths on both sides of the short / medium / long classes, empty rows, tails of every width; the wide X takes
    the tiles of 64 floats."""
    lens = np.array([0, 1, 7, 8, 9, 31, 32, 33, 64, 65, 511, 512, 513, 1025, 2999])
    deg = np.random.default_rng(feat).choice(lens, n_rows)
    deg[-1] = 2999                                             # a long row in the last, partly filled workgroup
    w = workloads.random_csr(n_rows, n_cols, deg, 40 + feat, feat)
    d = upload(w)
    Y = torch.full((n_rows, feat), float("nan"), device="cuda")
    gpu_lib.sptir_spmm_csr(w.n_rows, w.n_cols, d.indptr, d.indices, d.values, d.X, Y)
    Yr, Sr = oracle.spmm_csr(w.n_rows, w.indptr, w.indices, w.values, w.X)
    assert_y_close(Y.cpu().numpy(), Yr, Sr, what=f"rows={n_rows} cols={n_cols} feat={feat}")


@pytest.mark.parametrize("n_rows,feat,mean", [(200, 3, 20), (200, 17, 20), (129, 36, 20), (1000, 130, 20),   # 64 rows a workgroup
                                              (8200, 3, 45), (8193, 16, 45), (2049, 160, 60), (2050, 161, 60),   # 16
                                              (90, 40, 60), (89, 5, 60)])                                        # 8
def test_rows_per_workgroup(gpu_lib, n_rows, feat, mean):
    """Row classes in workgroups of 64, 16 and 8 rows, the last one partly filled."""
    rng = np.random.default_rng(feat)
    deg = rng.integers(0, 2 * mean, n_rows)
    some = rng.choice(n_rows, 8, replace=False)
    deg[some] = [0, 32, 33, 256, 257, 512, 513, 300]
    deg[:] = np.minimum(deg, 700)
    w = workloads.random_csr(n_rows, 700, deg, feat, feat)
    d = upload(w)
    Y = torch.full((n_rows, feat), float("nan"), device="cuda")
    gpu_lib.sptir_spmm_csr(w.n_rows, w.n_cols, d.indptr, d.indices, d.values, d.X, Y)
    Yr, Sr = oracle.spmm_csr(w.n_rows, w.indptr, w.indices, w.values, w.X)
    assert_y_close(Y.cpu().numpy(), Yr, Sr, what=f"rows={n_rows} feat={feat} mean={mean}")


@pytest.mark.parametrize("n_rows,feat", [(1, 4), (511, 3), (513, 16), (1025, 41), (6000, 67), (40_000, 36), (17_000, 1028)])
def test_long_rows_among_short_ones(gpu_lib, n_rows, feat):
    """Rows of a few entries, whose long ones workgroups of their own take: none, one in the last row, several next to each
    other, more rows than those workgroups look through at a time."""
    rng = np.random.default_rng(n_rows)
    deg = rng.integers(0, 6, n_rows)
    if n_rows > 500:
        at = np.r_[n_rows - 1, 63, 64, 65, rng.choice(n_rows - 1, min(12, n_rows // 400), replace=False)]
        deg[at] = rng.choice([512, 513, 600, 1100], at.size)
    w = workloads.random_csr(n_rows, 1200, deg, feat, feat)
    d = upload(w)
    Y = torch.full((n_rows, feat), float("nan"), device="cuda")
    gpu_lib.sptir_spmm_csr(w.n_rows, w.n_cols, d.indptr, d.indices, d.values, d.X, Y)
    Yr, Sr = oracle.spmm_csr(w.n_rows, w.indptr, w.indices, w.values, w.X)
    assert_y_close(Y.cpu().numpy(), Yr, Sr, what=f"rows={n_rows} feat={feat}")


@pytest.mark.parametrize("n_rows,feat", [(129, 4), (4000, 13), (20_000, 64), (70_000, 36), (3000, 1028)])
def test_long_rows_that_are_neighbours(gpu_lib, n_rows, feat):
    """Rows in the order of their lengths: those workgroups that take the long rows each have some of them, and all are taken once."""
    rng = np.random.default_rng(n_rows)
    deg = rng.integers(0, 6, n_rows)
    deg[:n_rows // 400 + 1] = rng.choice([512, 513, 600, 1100], n_rows // 400 + 1)
    deg = np.sort(deg)[::-1] if n_rows % 3 else np.sort(deg)
    w = workloads.random_csr(n_rows, 1200, deg, feat, feat)
    assert w.nnz < 24 * n_rows
    d = upload(w)
    Y = torch.full((n_rows, feat), float("nan"), device="cuda")
    gpu_lib.sptir_spmm_csr(w.n_rows, w.n_cols, d.indptr, d.indices, d.values, d.X, Y)
    Yr, Sr = oracle.spmm_csr(w.n_rows, w.indptr, w.indices, w.values, w.X)
    assert_y_close(Y.cpu().numpy(), Yr, Sr, what=f"rows={n_rows} feat={feat}")
