"""Rows of a hyb handle that are summed from column slices in LDS: which rows those are, that none of their entries is left in the
stream, and Y against the fp64 oracle (|Y - Y_oracle| <= 1e-5 * sum_j |a_ij x_jk|, exactly 0 where that is 0)."""
import numpy as np
import pytest
import torch

import oracle
import workloads
from gpu_helpers import fetch_hyb, upload
from hyb_checks import assert_same_hyb
from test_gpu_parity import assert_y_close, say
from test_gpu_stream import decode

pytestmark = pytest.mark.gpu
SLICE, PIECE, LEAST = 2496, 8, 64     # columns of a slice, entries per slice and entries from which on a row is long
ERR_ALLOC = 4


def matrix(n_rows, n_cols, n_long, feat, seed, one_value):
    """n_long rows from the shortest long one to a full one, the others just too short, empty, or of a few entries."""
    rng = np.random.default_rng(seed)
    least = max(LEAST, PIECE * n_cols // SLICE)
    deg = rng.integers(0, 9, n_rows)
    at = rng.permutation(n_rows)
    deg[at[:n_long]] = np.minimum(n_cols, (least * rng.uniform(1.0, 6.0, n_long)).astype(np.int64))
    deg[at[0]], deg[at[n_long - 1]] = n_cols, min(n_cols, least)
    deg[at[n_long:n_long + 3]] = min(n_cols, least - 1)
    w = workloads.random_csr(n_rows, n_cols, deg, seed, feat)
    if one_value:
        w.values[:] = np.repeat(rng.standard_normal(n_rows).astype(np.float32), np.diff(w.indptr))
    return w, np.flatnonzero(deg >= least)


@pytest.mark.parametrize("n_rows,n_cols,n_long", [(40, 100, 1), (70, 2495, 16), (300, 2496, 17), (300, 2497, 33),
                                                  (2700, 5200, 2300), (700, 30001, 260)])
@pytest.mark.parametrize("feat", [1, 3, 4, 7, 16, 17, 41, 64, 128, 131])
@pytest.mark.parametrize("one_value", [False, True])
def test_long_rows(gpu_lib, n_rows, n_cols, n_long, feat, one_value):
    sptir = gpu_lib
    say(f"[long rows] {n_rows}x{n_cols} long={n_long} feat={feat} one_value={one_value}")
    w, long_rows = matrix(n_rows, n_cols, n_long, feat, n_cols + feat, one_value)
    d = upload(w)
    Yr, Sr = oracle.spmm_csr(w.n_rows, w.indptr, w.indices, w.values, w.X)
    for c, options in ((3, {"column_slices": 1, "rounds": 1}), (2, {"column_slices": 1, "rounds": 2, "parts_per_launch": 1}),
                       (1, {"column_slices": 1, "keep_values": 1, "feat_hint": 32})):
        hyb = sptir.sptir_hyb_build_ex(n_rows, n_cols, d.indptr, d.indices, d.values, c, 5, options)
        rows = sptir.sptir_hyb_array(hyb, "plan_long_rows")
        lens = np.diff(w.indptr)[rows]
        assert np.array_equal(np.sort(rows), long_rows)
        assert (lens <= 1.03 * np.minimum.accumulate(lens)).all(), "longest first, up to a class of length"
        Y = torch.full((n_rows, feat), float("nan"), device="cuda")
        sptir.sptir_spmm(hyb, d.X, Y)
        assert_y_close(Y.cpu().numpy(), Yr, Sr, what=f"{options}")
        again = torch.full_like(Y, float("nan"))
        sptir.sptir_spmm_noalloc(hyb, d.X, again)
        assert torch.equal(Y, again)
        hyb.destroy()


@pytest.mark.parametrize("options", [{"rounds": 1}, {"rounds": 2, "wide_stream": 1, "heavy_len": 20}])
def test_long_rows_leave_the_stream_and_nothing_else(gpu_lib, options):
    sptir = gpu_lib
    w, long_rows = matrix(400, 3000, 40, 4, 9, False)
    d = upload(w)
    hyb = sptir.sptir_hyb_build_ex(w.n_rows, w.n_cols, d.indptr, d.indices, d.values, 3, 4, {**options, "column_slices": 1})
    got, info = fetch_hyb(sptir, hyb)
    assert_same_hyb(got, oracle.hyb_build(w.n_rows, w.n_cols, w.indptr, w.indices, w.values, 3, 4))
    assert info["n_heavy_pieces"] >= long_rows.size
    in_long = int(np.diff(w.indptr)[long_rows].sum())
    assert info["n_heavy_nnz"] >= in_long
    sequence = dict(info, n_heavy_pieces=info["n_heavy_pieces"] - long_rows.size)
    rows, cols, vals = decode(sptir, hyb, sequence, w)
    want_rows = np.repeat(np.arange(w.n_rows, dtype=np.int64), np.diff(w.indptr))
    keep = ~np.isin(want_rows, long_rows)
    o = np.argsort(rows * w.n_cols + cols, kind="stable")
    assert np.array_equal((rows * w.n_cols + cols)[o], (want_rows * w.n_cols + w.indices)[keep])
    assert np.array_equal(vals[o], w.values.view(np.int32).astype(np.int64)[keep])


@pytest.mark.parametrize("one_value", [False, True])
def test_rows_of_x_that_are_not_finite_stay_with_their_rows(gpu_lib, one_value):
    sptir = gpu_lib
    w, long_rows = matrix(200, 4000, 150, 20, 3, one_value)
    w.X[17, 3] = np.inf; w.X[2495, 0] = np.nan; w.X[3999, 19] = -np.inf
    d = upload(w)
    hyb = sptir.sptir_hyb_build_ex(w.n_rows, w.n_cols, d.indptr, d.indices, d.values, 1, 5, {"column_slices": 1, "rounds": 2})
    Y = torch.empty(w.n_rows, 20, device="cuda")
    sptir.sptir_spmm(hyb, d.X, Y)
    got = np.isfinite(Y.cpu().numpy())
    rows = np.repeat(np.arange(w.n_rows), np.diff(w.indptr))
    want = np.ones((w.n_rows, 20), bool)
    for col, f in ((17, 3), (2495, 0), (3999, 19)):
        want[rows[w.indices == col], f] = False
    assert np.array_equal(got[long_rows], want[long_rows])


def large_matrix(n_rows, share, n_cols=40000, n_groups=10, deg=1600, feat=8, one_range=False):
    """Rows of like length, a few longer; `share` of a row's entries in one of n_groups ranges of columns (the same one for all
    rows, or its own), the others anywhere."""
    rng = np.random.default_rng(n_rows)
    lens = rng.integers(deg - 60, deg, n_rows)
    lens[rng.choice(n_rows, 5, replace=False)] = 5 * deg
    width = n_cols // n_groups
    inside = np.minimum((share * lens).astype(np.int64), width * 7 // 8)
    a = workloads.random_csr(n_rows, width, inside, 1, feat)
    b = workloads.random_csr(n_rows, n_cols, lens - inside, 2, feat)
    row_of = lambda w: np.repeat(np.arange(n_rows, dtype=np.int64), np.diff(w.indptr))
    ra, rb = row_of(a), row_of(b)
    key = np.unique(np.concatenate([ra * n_cols + (0 if one_range else ra % n_groups * width) + a.indices, rb * n_cols + b.indices]))
    rows = key // n_cols
    w = b
    w.indptr = np.concatenate([[0], np.cumsum(np.bincount(rows, minlength=n_rows))]).astype(np.int32)
    w.indices = (key - rows * n_cols).astype(np.int32)
    w.values = rng.standard_normal(key.size).astype(np.float32)
    return w


def build_and_multiply(sptir, w, d, options):
    hyb = sptir.sptir_hyb_build_ex(w.n_rows, w.n_cols, d.indptr, d.indices, d.values, 2, 7, options)
    Y = torch.full((w.n_rows, w.X.shape[1]), float("nan"), device="cuda")
    sptir.sptir_spmm(hyb, d.X, Y)
    info, n_long = sptir.sptir_hyb_info(hyb), sptir.sptir_hyb_array(hyb, "plan_long_rows").size
    hyb.destroy()
    return Y, info, n_long


@pytest.mark.parametrize("share", [0.0, 0.3, 0.8])
def test_slices_only_where_a_block_of_rows_is_alike(gpu_lib, share):
    """Where rows have their entries in ranges of their own, a block's steps are those of a different row in every slice:
    such a graph is built as without column slices, unless they are asked for."""
    sptir = gpu_lib
    w = large_matrix(9000, share)
    say(f"[long rows] share={share} nnz={w.indices.size}")
    assert w.indices.size > 12_700_000
    d = upload(w)
    Yr, Sr = oracle.spmm_csr(w.n_rows, w.indptr, w.indices, w.values, w.X)
    sptir.sptir_release_scratch()
    plain, plain_info, none = build_and_multiply(sptir, w, d, {"column_slices": 2})
    assert none == 0
    sptir.sptir_release_scratch()
    Y, info, n_long = build_and_multiply(sptir, w, d, {})
    assert_y_close(Y.cpu().numpy(), Yr, Sr, what=f"share {share}")
    if share == 0:
        assert n_long == w.n_rows
    else:
        assert n_long == 0 and torch.equal(Y, plain)
        assert {k: v for k, v in info.items() if k != "device_bytes"} == \
               {k: v for k, v in plain_info.items() if k != "device_bytes"}
        assert info["device_bytes"] <= 1.3 * plain_info["device_bytes"]      # (a kept block counts whole, up to a quarter larger)
    Y, _, n_long = build_and_multiply(sptir, w, d, {"column_slices": 1})
    assert n_long == w.n_rows
    assert_y_close(Y.cpu().numpy(), Yr, Sr, what=f"share {share}, asked for")


def test_few_long_entries_stay_in_the_stream(gpu_lib):
    """A build and one product of so few entries take longer with column slices: they are left to callers who ask."""
    w = large_matrix(5000, 0.0)
    assert 6_000_000 < w.indices.size < 12_500_000
    d = upload(w)
    assert build_and_multiply(gpu_lib, w, d, {})[2] == 0
    assert build_and_multiply(gpu_lib, w, d, {"column_slices": 1})[2] == w.n_rows


def test_slices_that_find_no_memory_are_left_out(gpu_lib):
    """An allocation that only column slices ask for may fail: the build then does without them, unless the caller asked for
    them.  (A caller's allocator that refuses one size, an error code and no GPU work.)"""
    import ctypes
    from paper_2207_04606_amd import binding
    sptir = gpu_lib
    w = large_matrix(9000, 0.0)
    d = upload(w)
    asked, refuse = [], set()

    @binding._ALLOC_FN
    def take(nbytes, ctx, stream):
        asked.append(int(nbytes))
        return None if int(nbytes) in refuse else binding._torch_alloc(nbytes, ctx, stream)

    lib = sptir.load_library()
    assert lib.sptir_set_allocator(take, binding._torch_free, None) == 0
    try:
        plain, _, _ = build_and_multiply(sptir, w, d, {"column_slices": 2})
        without = set(asked)
        asked.clear()
        _, _, n_long = build_and_multiply(sptir, w, d, {})
        assert n_long == w.n_rows
        only = sorted(set(asked) - without, key=asked.index)[:2]   # the counts of steps, the handle's arrays of slices
        assert len(only) == 2
        before = len(binding._torch_blocks)
        for size in only:
            refuse = {size}
            Y, _, n_long = build_and_multiply(sptir, w, d, {})
            assert n_long == 0 and torch.equal(Y, plain), size
            with pytest.raises(sptir.SptirError) as e:
                build_and_multiply(sptir, w, d, {"column_slices": 1})
            assert e.value.status == ERR_ALLOC
        assert len(binding._torch_blocks) == before, "a build that failed keeps memory"
    finally:
        sptir.sptir_set_allocator(False)


@pytest.mark.parametrize("share,sliced", [(0.1, True), (0.6, False)])
def test_slices_only_where_none_is_much_hotter_than_the_mean(gpu_lib, share, sliced):
    """Entries in one range of columns: panels as small as it takes for all CUs to have some of the hot slice, and no slices where
    it has more than 16 times the mean's entries, unless they are asked for."""
    w = large_matrix(9000, share, n_cols=82000, n_groups=34, one_range=True)
    say(f"[long rows] hot share={share} nnz={w.indices.size}")
    assert w.indices.size > 12_700_000
    d = upload(w)
    Yr, Sr = oracle.spmm_csr(w.n_rows, w.indptr, w.indices, w.values, w.X)
    Y, _, n_long = build_and_multiply(gpu_lib, w, d, {})
    assert n_long == (w.n_rows if sliced else 0)
    assert_y_close(Y.cpu().numpy(), Yr, Sr, what=f"hot share {share}")
    if not sliced:
        assert torch.equal(Y, build_and_multiply(gpu_lib, w, d, {"column_slices": 2})[0])
        Y, _, n_long = build_and_multiply(gpu_lib, w, d, {"column_slices": 1})
        assert n_long == w.n_rows
        assert_y_close(Y.cpu().numpy(), Yr, Sr, what=f"hot share {share}, asked for")
