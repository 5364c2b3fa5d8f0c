"""Chunk lists that several wavefronts of a workgroup share (small matrices with a long list): the ranges end inside queue chunks
and inside rows that all lane groups share, at lists of every number of quads, in both record forms and with and without values."""
import numpy as np
import pytest
import torch

import oracle
import workloads
from gpu_helpers import upload
from test_gpu_parity import assert_y_close, say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("feat", [1, 3, 4, 16, 17, 32, 41, 64, 100])
@pytest.mark.parametrize("one_value", [False, True])
@pytest.mark.parametrize("wide", [0, 1])
def test_shared_lists(gpu_lib, feat, one_value, wide):
    for n_rows, n_cols, kind in ((1, 300, "rows"), (9, 2100, "rows"), (300, 2100, "rows"), (500, 900, "even"), (2000, 900, "even"),
                                 (700, 6000, "one"),
                                 (300, 165_000, "rows"), (900, 165_000, "even")):   # 16 lanes a group from 41 features on
        if n_cols > 100_000 and feat not in (41, 100):
            continue
        say(f"[shared lists] feat={feat} one_value={one_value} wide={wide} {n_rows}x{n_cols} {kind}")
        rng = np.random.default_rng(n_rows + feat)
        deg = rng.integers(0, 9, n_rows)
        if kind == "rows":       # lists of 2, 3, .. quads through a row of 257, 513, .. entries; the rows around it short
            at = np.arange(0, n_rows, 8)
            deg[at] = np.minimum(n_cols, 256 * rng.integers(0, 8, at.size) + rng.integers(1, 40, at.size))
            deg[-1] = min(n_cols, 257)
        elif kind == "even":     # queues of every length
            deg = rng.integers(20, 120, n_rows)
        else:
            deg[n_rows // 2] = 2047
        w = workloads.random_csr(n_rows, n_cols, deg, feat, feat)
        if one_value:
            w.values[:] = np.repeat(rng.standard_normal(n_rows).astype(np.float32), np.diff(w.indptr))
        d = upload(w)
        Yr, Sr = oracle.spmm_csr(w.n_rows, w.indptr, w.indices, w.values, w.X)
        for c, k in ((1, 3), (3, 11)):
            hyb = gpu_lib.sptir_hyb_build_ex(n_rows, n_cols, d.indptr, d.indices, d.values, c, k,
                                             {"wide_stream": wide, "heavy_len": 2048, "rounds": 2})
            Y = torch.full((n_rows, feat), float("nan"), device="cuda")
            gpu_lib.sptir_spmm(hyb, d.X, Y)
            assert_y_close(Y.cpu().numpy(), Yr, Sr, what=f"{n_rows}x{n_cols} {kind} c={c}")
            timed = torch.full_like(Y, float("nan"))
            times = gpu_lib.sptir_spmm_timed(hyb, d.X, timed)
            assert torch.equal(Y, timed)
            several_launches = n_cols > 100_000 and c == 3
            assert (times["list_waves"] > 1) != several_launches and times["list_waves"] <= 8
            assert times["tile_floats"] == (64 if n_cols > 100_000 else 32 if feat > 16 else 16 if feat >= 4 else 4)
            again = torch.full_like(Y, float("nan"))
            gpu_lib.sptir_spmm_noalloc(hyb, d.X, again)
            assert torch.equal(Y, again)
            hyb.destroy()


@pytest.mark.parametrize("feat", [1, 4, 17, 41, 64])
@pytest.mark.parametrize("long_list", [False, True])
def test_lists_to_share_beside_heavy_ones(gpu_lib, feat, long_list):
    """A list of 8 quads among lists of one is shared, and heavy lists then have a launch of their own; lists that are all short are in
    the heavy lists' launch, each for one wavefront.  More heavy lists than chunk lists, and fewer."""
    for n_rows, n_heavy in ((700, 3), (100, 60)):
        say(f"[shared beside heavy] feat={feat} long_list={long_list} {n_rows} rows, {n_heavy} heavy")
        rng = np.random.default_rng(n_rows + feat)
        deg = rng.integers(1, 9, n_rows)
        deg[:n_heavy] = rng.integers(2049, 2400, n_heavy)
        if long_list:
            deg[n_rows // 2 + 20] = 2047
        w = workloads.random_csr(n_rows, 6000, deg, feat, feat)
        d = upload(w)
        Yr, Sr = oracle.spmm_csr(w.n_rows, w.indptr, w.indices, w.values, w.X)
        hyb = gpu_lib.sptir_hyb_build_ex(n_rows, 6000, d.indptr, d.indices, d.values, 1, 11, {"heavy_len": 2048, "rounds": 2,
                                                                                           "column_slices": 2})
        assert gpu_lib.sptir_hyb_info(hyb)["n_heavy_pieces"] == n_heavy
        Y = torch.full((n_rows, feat), float("nan"), device="cuda")
        gpu_lib.sptir_spmm(hyb, d.X, Y)
        assert_y_close(Y.cpu().numpy(), Yr, Sr, what=f"{n_rows} rows, {n_heavy} heavy")
        timed = torch.full_like(Y, float("nan"))
        assert (gpu_lib.sptir_spmm_timed(hyb, d.X, timed)["list_waves"] > 1) == long_list
        assert torch.equal(Y, timed)
        again = torch.full_like(Y, float("nan"))
        gpu_lib.sptir_spmm_noalloc(hyb, d.X, again)
        assert torch.equal(Y, again)
        hyb.destroy()
