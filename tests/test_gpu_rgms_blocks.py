"""RGMS with blocks of any number of rows (csrc/rgms_blocks.h): Y against the fp64 oracle."""
import numpy as np
import pytest

import oracle
import workloads
from test_gpu_parity import say
from test_gpu_rgms import assert_y_close, run_rgms

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d_out", [64, 128, 256])
@pytest.mark.parametrize("n,mean,rows", [(128 * 320, 0.3, 160), (128 * 321, 0.3, 81), (64 * 318, 0.6, 80), (32 * 319, 1.2, 40), (128 * 530, 0.3, 133), (128 * 576, 0.3, 144), (128 * 577, 0.3, 97),
                                         (64 * 300, 0.6, 75), (64 * 570 + 3, 0.6, 72), (32 * 280, 1.2, 35), (32 * 321, 1.2, 21), (32 * 570, 1.2, 36), (32 * 936, 1.2, 39),
                                         (64 * 1230, 0.6, 77), (32 * 1249, 1.2, 32), (512 * 192, 0.03, 384), (512 * 200 + 3, 0.03, 401),
                                         (512 * 255 - 1, 0.03, 510)])
def test_rgms_columns_beside_blocks_of_any_rows(gpu_lib, n, mean, rows, d_out):
    """Blocks that have grown past a power of two rows keep its columns of Y per pass, those of 512 rows have become fewer; at the ends of
    the ranges in which they do."""
    say(f"[rgms columns] {n} rows d_out={d_out}")
    n_rel, d_in = 3, 32
    rng = np.random.default_rng(n + d_out)
    w = workloads.random_csr(n_rel * n, n, rng.poisson(mean, n_rel * n), 1, 1)
    X = rng.standard_normal((n, d_in)).astype(np.float32)
    W = rng.standard_normal((n_rel, d_in, d_out)).astype(np.float32)
    w = workloads.HeteroWorkload("columns", n, n_rel, w.indptr, w.indices, w.values, X, W)
    Y, info = run_rgms(gpu_lib, w)
    assert info["row_block"] == rows
    Yr, Sr = oracle.rgms(n_rel, n, w.indptr, w.indices, w.values, w.X, w.W)
    assert_y_close(Y, Yr, Sr, f"{n} rows")
