"""GPU parity tests of SDDMM on CSR: through the C ABI, against the fp64 oracle.
Criterion: |B_gpu - B_oracle| <= 1e-5 * |a_ij| * sum_k |x_ik y_kj| per entry (fp32 products and a d-term sum
against fp64: the error is a few u * sqrt(d) of that magnitude sum, u = 2^-24), and exactly 0 where it is 0."""
import numpy as np
import pytest
import torch

import oracle
import workloads
from test_gpu_parity import ragged_workload, say

pytestmark = pytest.mark.gpu
B_TOL = 1e-5


def run_sddmm(sptir, w, Xr, Yt, in_place=False):
    dev = "cuda"
    ip = torch.from_numpy(w.indptr).to(dev)
    ix = torch.from_numpy(w.indices).to(dev)
    va = torch.from_numpy(w.values).to(dev)
    B = va if in_place else torch.full((w.nnz,), float("nan"), device=dev)
    sptir.sptir_sddmm_csr(w.n_rows, w.n_cols, ip, ix, va, torch.from_numpy(Xr).to(dev), torch.from_numpy(Yt).to(dev), B)
    return B.cpu().numpy()


def assert_b_close(B_gpu, B_ref, M_ref, what):
    B_gpu = B_gpu.astype(np.float64)
    assert np.isfinite(B_gpu).all(), f"{what}: non-finite output"
    zero = M_ref == 0
    assert (B_gpu[zero] == 0).all(), what
    ratio = np.abs(B_gpu - B_ref)[~zero] / M_ref[~zero]
    worst = float(ratio.max()) if ratio.size else 0.0
    assert worst <= B_TOL, f"{what}: max normalised error {worst:.3e}"
    return worst


def left_operand(w, feat, seed):
    return np.random.default_rng(seed).standard_normal((w.n_rows, feat)).astype(np.float32)


@pytest.mark.parametrize("feat", [1, 3, 4, 8, 28, 32, 36, 64, 100, 128, 132, 256, 260, 512, 516, 640])
def test_sddmm_feature_widths(gpu_lib, feat):
    say(f"[sddmm feat] feat={feat}")
    w = ragged_workload(700 + feat, 1300, 1100, feat, max_deg=700, long_rows=5)
    Xr = left_operand(w, feat, feat)
    B = run_sddmm(gpu_lib, w, Xr, w.X)
    Br, Mr = oracle.sddmm_csr(w.n_rows, w.indptr, w.indices, w.values, Xr, w.X)
    assert_b_close(B, Br, Mr, f"feat={feat}")


def test_sddmm_in_place_and_repeatable(gpu_lib):
    w = ragged_workload(41, 900, 1000, 64, max_deg=500, long_rows=3)
    Xr = left_operand(w, 64, 1)
    B1 = run_sddmm(gpu_lib, w, Xr, w.X)
    B2 = run_sddmm(gpu_lib, w, Xr, w.X, in_place=True)     # B written over A's values
    assert np.array_equal(B1, B2)


def test_sddmm_many_empty_rows_and_tiny_inputs(gpu_lib):
    # mostly empty rows: the row of an entry is found by walking indptr
    rng = np.random.default_rng(5)
    deg = np.zeros(5000, dtype=np.int64)
    deg[rng.choice(5000, 40, replace=False)] = rng.integers(1, 300, 40)
    w = workloads.random_csr(5000, 700, deg, 5, 32)
    Xr = left_operand(w, 32, 2)
    Br, Mr = oracle.sddmm_csr(w.n_rows, w.indptr, w.indices, w.values, Xr, w.X)
    assert_b_close(run_sddmm(gpu_lib, w, Xr, w.X), Br, Mr, "empty rows")
    # one entry; and no entries at all (nothing is launched)
    w1 = workloads.random_csr(3, 4, np.array([0, 1, 0]), 1, 8)
    X1 = left_operand(w1, 8, 3)
    Br, Mr = oracle.sddmm_csr(3, w1.indptr, w1.indices, w1.values, X1, w1.X)
    assert_b_close(run_sddmm(gpu_lib, w1, X1, w1.X), Br, Mr, "single entry")
    w0 = workloads.random_csr(3, 4, np.array([0, 0, 0]), 1, 8)
    assert run_sddmm(gpu_lib, w0, left_operand(w0, 8, 4), w0.X).shape == (0,)


def test_sddmm_closed_forms(gpu_lib):
    w = ragged_workload(43, 600, 800, 128, max_deg=300, long_rows=2)
    ones_r, ones_c = np.ones((w.n_rows, 128), np.float32), np.ones((w.n_cols, 128), np.float32)
    assert np.array_equal(run_sddmm(gpu_lib, w, ones_r, ones_c), 128.0 * w.values)      # exact in fp32
    rng = np.random.default_rng(3)
    lab_r, lab_c = rng.integers(0, 128, w.n_rows), rng.integers(0, 128, w.n_cols)
    B = run_sddmm(gpu_lib, w, np.eye(128, dtype=np.float32)[lab_r], np.eye(128, dtype=np.float32)[lab_c])
    rows = np.repeat(np.arange(w.n_rows), np.diff(w.indptr))
    assert np.array_equal(B, np.where(lab_r[rows] == lab_c[w.indices], w.values, np.float32(0)))


def test_sddmm_unaligned_views(gpu_lib):
    w = ragged_workload(47, 300, 350, 12, max_deg=200, long_rows=2)
    Xr = left_operand(w, 12, 5)
    Br, Mr = oracle.sddmm_csr(w.n_rows, w.indptr, w.indices, w.values, Xr, w.X)
    dev = "cuda"
    ip, ix, va = (torch.from_numpy(a).to(dev) for a in (w.indptr, w.indices, w.values))
    for shift in (1, 2):
        xb = torch.empty(Xr.size + 4, device=dev)
        yb = torch.empty(w.X.size + 4, device=dev)
        X = xb[shift:shift + Xr.size].view(w.n_rows, 12); X.copy_(torch.from_numpy(Xr))
        Y = yb[shift:shift + w.X.size].view(w.n_cols, 12); Y.copy_(torch.from_numpy(w.X))
        B = torch.full((w.nnz,), float("nan"), device=dev)
        gpu_lib.sptir_sddmm_csr(w.n_rows, w.n_cols, ip, ix, va, X, Y, B)
        assert_b_close(B.cpu().numpy(), Br, Mr, f"shift={shift}")


def test_sddmm_error_paths(gpu_lib):
    w = ragged_workload(48, 50, 60, 8, max_deg=20)
    dev = "cuda"
    ip, ix, va = (torch.from_numpy(a).to(dev) for a in (w.indptr, w.indices, w.values))
    X = torch.zeros(w.n_rows, 8, device=dev); Y = torch.zeros(w.n_cols, 8, device=dev)
    with pytest.raises(ValueError):
        gpu_lib.sptir_sddmm_csr(w.n_rows, w.n_cols, ip, ix, va, X, Y[:, :4].contiguous(), torch.empty(w.nnz, device=dev))
    with pytest.raises(ValueError):
        gpu_lib.sptir_sddmm_csr(w.n_rows, w.n_cols, ip, ix, va, X, Y, torch.empty(w.nnz + 1, device=dev))
    with pytest.raises(gpu_lib.SptirError):      # B overlapping a dense operand
        gpu_lib.sptir_sddmm_csr(w.n_rows, w.n_cols, ip, ix, va, X, Y, X.view(-1)[:w.nnz])


@pytest.mark.parametrize("name", ["tiny", "small", "medium", "protein", "social"])
def test_sddmm_named_configs(gpu_lib, name):
    w = workloads.make_config(name, feat=128 if name == "social" else None)
    say(f"[sddmm config] {name} nnz={w.nnz} feat={w.feat}")
    Xr = left_operand(w, w.feat, 9)
    B = run_sddmm(gpu_lib, w, Xr, w.X)
    Br, Mr = oracle.sddmm_csr(w.n_rows, w.indptr, w.indices, w.values, Xr, w.X)
    worst = assert_b_close(B, Br, Mr, name)
    say(f"[sddmm config] {name}: max_err={worst:.2e}")


def run_sddmm_plan(sptir, w, Xr, Yt, c, feat_hint=0, in_place=False):
    dev = "cuda"
    ip = torch.from_numpy(w.indptr).to(dev)
    ix = torch.from_numpy(w.indices).to(dev)
    va = torch.from_numpy(w.values).to(dev)
    plan = sptir.sptir_sddmm_plan_build(w.n_rows, w.n_cols, ip, ix, c, feat_hint)
    info = sptir.sptir_sddmm_plan_info(plan)
    B = va if in_place else torch.full((w.nnz,), float("nan"), device=dev)
    sptir.sptir_sddmm(plan, va, torch.from_numpy(Xr).to(dev), torch.from_numpy(Yt).to(dev), B)
    out = B.cpu().numpy()
    plan.destroy()
    return out, info


@pytest.mark.parametrize("c", [1, 2, 3, 8, 16, 40, 2000])
@pytest.mark.parametrize("feat", [4, 32, 100, 128, 7])
def test_sddmm_with_plan_equals_csr_order(gpu_lib, c, feat):
    """Partition order changes where an entry is computed, not how: the plan path must give the very bits of the
    CSR-order kernel (same per-entry arithmetic), for any number of partitions including more than columns."""
    say(f"[sddmm plan] c={c} feat={feat}")
    w = ragged_workload(800 + feat, 1300, 1100, feat, max_deg=700, long_rows=5)
    Xr = left_operand(w, feat, feat)
    want = run_sddmm(gpu_lib, w, Xr, w.X)
    got, info = run_sddmm_plan(gpu_lib, w, Xr, w.X, c)
    assert info["n_col_parts"] == min(c, w.n_cols) and info["nnz"] == w.nnz
    assert np.array_equal(got, want)
    Br, Mr = oracle.sddmm_csr(w.n_rows, w.indptr, w.indices, w.values, Xr, w.X)
    assert_b_close(got, Br, Mr, f"plan c={c} feat={feat}")


def test_sddmm_plan_edge_cases(gpu_lib):
    dev = "cuda"
    # no entries
    w0 = workloads.random_csr(3, 4, np.array([0, 0, 0]), 1, 8)
    got, info = run_sddmm_plan(gpu_lib, w0, left_operand(w0, 8, 4), w0.X, 2)
    assert got.shape == (0,) and info["nnz"] == 0
    # in place, automatic partition count, repeatable
    w = ragged_workload(49, 2000, 2500, 64, max_deg=1200, long_rows=10)
    Xr = left_operand(w, 64, 1)
    a, info = run_sddmm_plan(gpu_lib, w, Xr, w.X, 0, feat_hint=64)
    b, _ = run_sddmm_plan(gpu_lib, w, Xr, w.X, 0, feat_hint=64, in_place=True)
    assert np.array_equal(a, b) and info["n_col_parts"] in (1,) + tuple(range(8, 1025, 8))
    with pytest.raises(gpu_lib.SptirError):       # negative partition count
        gpu_lib.sptir_sddmm_plan_build(w.n_rows, w.n_cols, torch.from_numpy(w.indptr).to(dev),
                                       torch.from_numpy(w.indices).to(dev), -1)


@pytest.mark.parametrize("name", ["medium", "protein", "social"])
def test_sddmm_plan_named_configs(gpu_lib, name):
    w = workloads.make_config(name, feat=128)
    Xr = left_operand(w, 128, 9)
    B, info = run_sddmm_plan(gpu_lib, w, Xr, w.X, 0, feat_hint=128)
    say(f"[sddmm plan config] {name}: c={info['n_col_parts']} runs={info['n_runs']} bytes={info['device_bytes']}")
    Br, Mr = oracle.sddmm_csr(w.n_rows, w.indptr, w.indices, w.values, Xr, w.X)
    assert_b_close(B, Br, Mr, name)


@pytest.mark.parametrize("feat", [2, 5, 33, 63, 96, 160, 224, 257, 300])
@pytest.mark.parametrize("gap", [0, 1, 90, 700])
def test_sddmm_rows_of_a_chunk_and_row_ends(gpu_lib, gap, feat):
    """Chunks of 64 entries inside one row, over rows of one entry, and over more than 64 rows at a time (`gap` empty rows
    after each), with rows of X and Yt that end anywhere in a lane's four floats; in CSR order and with a plan."""
    say(f"[sddmm rows] gap={gap} feat={feat}")
    deg = np.concatenate([[200], np.tile(np.r_[[1], np.zeros(gap, dtype=int)], 150), [0, 63, 64, 65, 1, 1]])
    w = workloads.random_csr(deg.size, 900, deg, feat + gap, feat)
    Xr = left_operand(w, feat, 5)
    Br, Mr = oracle.sddmm_csr(w.n_rows, w.indptr, w.indices, w.values, Xr, w.X)
    assert_b_close(run_sddmm(gpu_lib, w, Xr, w.X), Br, Mr, f"gap={gap} feat={feat}")
    assert_b_close(run_sddmm_plan(gpu_lib, w, Xr, w.X, 8)[0], Br, Mr, f"plan gap={gap} feat={feat}")


@pytest.mark.parametrize("feat", [96, 97, 100, 127, 128, 129])
@pytest.mark.parametrize("past", [0, 1])
def test_sddmm_plan_lists_on_both_sides_of_l2(gpu_lib, past, feat):
    """Chunks of 64 entries of about 16 rows, of about 26 and of any number, all in one partition whose rows of Yt are 4 MB at most or
    one row more: with four float4 a lane other numbers of rows are staged there.  The bits are those of CSR order."""
    say(f"[sddmm L2] past={past} feat={feat}")
    width = (4 << 20) // (4 * feat) + past
    deg = np.concatenate([np.full(160, 4), np.tile([2, 3], 130), np.full(70, 64 // 15), np.random.default_rng(feat).integers(0, 9, 300)])
    w = workloads.random_csr(deg.size, width, deg, feat + past, feat)
    w.n_cols = 8 * width
    w.X = np.random.default_rng(past).standard_normal((w.n_cols, feat)).astype(np.float32)
    Xr = left_operand(w, feat, 3)
    got, info = run_sddmm_plan(gpu_lib, w, Xr, w.X, 8, feat_hint=feat)
    assert info["part_width"] == width and info["n_runs"] == -(-w.nnz // 512)
    assert np.array_equal(got, run_sddmm(gpu_lib, w, Xr, w.X))
    Br, Mr = oracle.sddmm_csr(w.n_rows, w.indptr, w.indices, w.values, Xr, w.X)
    assert_b_close(got, Br, Mr, f"past={past} feat={feat}")


def matrix_with_long_rows(n_rows, n_long, n_cols, seed, feat):
    rng = np.random.default_rng(seed)
    deg = rng.integers(0, 12, n_rows)
    at = rng.choice(n_rows, n_long, replace=False)
    deg[at] = rng.integers(n_cols // 2, n_cols, n_long)
    deg[at[:3]] = n_cols - 1, n_cols, n_cols // 8
    return workloads.random_csr(n_rows, n_cols, deg, seed, feat)


@pytest.mark.parametrize("hint,feat", [(36, 36), (41, 41), (64, 64), (96, 96), (97, 97), (128, 128), (131, 131), (160, 160), (192, 192),
                                       (224, 224), (250, 250), (255, 255), (256, 256),
                                       (128, 3), (128, 20), (128, 64), (128, 132), (128, 300),
                                       (253, 257), (256, 257), (256, 260), (256, 272), (256, 288), (256, 289)])
def test_sddmm_plan_takes_long_rows_in_column_slices(gpu_lib, hint, feat):
    """Rows with entries in every slice of columns, next to short and empty ones; pieces of full segments, of every
    remainder, and none; the last slice narrower; also calls with fewer and more features than the slices were made for."""
    say(f"[sddmm slices] hint={hint} feat={feat}")
    want_nnz = (1 << 29 if hint <= 64 or hint % 4 else 1 << 27) // hint     # (as many entries as the rule asks for)
    n_cols = 12001 if want_nnz > 2_000_000 else 3001
    n_long = want_nnz * 4 // (3 * n_cols) * 11 // 10 + 20
    w = matrix_with_long_rows(n_long + 300, n_long, n_cols, hint, feat)
    Xr = left_operand(w, feat, feat)
    want = run_sddmm(gpu_lib, w, Xr, w.X)
    got, info = run_sddmm_plan(gpu_lib, w, Xr, w.X, 8, feat_hint=hint)
    assert info["n_runs"] < 64, "the long rows are in the runs"
    assert np.array_equal(got, want)
    Br, Mr = oracle.sddmm_csr(w.n_rows, w.indptr, w.indices, w.values, Xr, w.X)
    assert_b_close(got, Br, Mr, f"hint={hint} feat={feat}")
    one_part, _ = run_sddmm_plan(gpu_lib, w, Xr, w.X, 1, feat_hint=hint, in_place=True)
    assert np.array_equal(one_part, want)


def test_sddmm_plan_slices_keep_non_finite_rows_apart(gpu_lib):
    """A row of X or Yt that is not finite reaches its own entries and no others, also past the end of a row that
    fills its lanes only in part."""
    n_long = 1100
    deg = np.random.default_rng(3).integers(11000, 13000, n_long)
    w = workloads.random_csr(n_long, 13500, deg, 3, 41)
    Xr = left_operand(w, 41, 1)
    Yt = w.X.copy()
    Xr[17, 40] = np.inf; Xr[18, 3] = np.nan; Yt[1999, 40] = np.nan; Yt[13499, 0] = -np.inf
    got, info = run_sddmm_plan(gpu_lib, w, Xr, Yt, 8, feat_hint=41)
    assert info["n_runs"] == 0
    rows = np.repeat(np.arange(n_long), deg)
    with np.errstate(invalid="ignore"):
        want = w.values * np.einsum("ij,ij->i", Xr[rows], Yt[w.indices])
    assert np.array_equal(np.isfinite(got), np.isfinite(want))


@pytest.mark.parametrize("feat", [96, 128, 256])
def test_sddmm_plan_slices_with_hot_columns(gpu_lib, feat):
    """Many entries in one slice of columns, whose work is dealt to several workgroups; rows without any there; short rows."""
    n_long, n_cols = 131072 // feat, 12001
    rng = np.random.default_rng(feat)
    far = workloads.random_csr(n_long + 50, n_cols - 130, np.r_[rng.integers(1000, 1300, n_long), rng.integers(0, 9, 50)], feat, feat)
    near = workloads.random_csr(n_long + 50, 130, np.r_[rng.integers(0, 131, n_long), np.zeros(50, dtype=int)], feat + 1, feat)
    rows = [np.repeat(np.arange(n_long + 50, dtype=np.int64), np.diff(m.indptr)) for m in (near, far)]
    key = np.sort(np.concatenate([rows[0] * n_cols + 5000 + near.indices,
                                  rows[1] * n_cols + np.where(far.indices < 5000, far.indices, far.indices + 130)]))
    w = near
    w.n_cols = n_cols
    w.indptr = np.concatenate([[0], np.cumsum(np.bincount(key // n_cols, minlength=n_long + 50))]).astype(np.int32)
    w.indices = (key % n_cols).astype(np.int32)
    w.values = rng.standard_normal(key.size).astype(np.float32)
    w.X = rng.standard_normal((n_cols, feat)).astype(np.float32)
    assert w.nnz * feat >= 1 << 27
    say(f"[sddmm hot columns] feat={feat} nnz={w.nnz}")
    Xr = left_operand(w, feat, feat)
    want = run_sddmm(gpu_lib, w, Xr, w.X)
    got, info = run_sddmm_plan(gpu_lib, w, Xr, w.X, 8, feat_hint=feat)
    assert info["n_runs"] < 16, "the long rows are in the runs"
    assert np.array_equal(got, want)
    Br, Mr = oracle.sddmm_csr(w.n_rows, w.indptr, w.indices, w.values, Xr, w.X)
    assert_b_close(got, Br, Mr, f"hot feat={feat}")


def test_sddmm_plan_lists_where_yt_is_near(gpu_lib):
    """Rows long enough for slices stay in the lists where Yt comes out of L2 as it is."""
    w = workloads.random_csr(9000, 9000, np.random.default_rng(7).integers(120, 300, 9000), 7, 128)
    assert w.nnz * 128 >= 1 << 27
    Xr = left_operand(w, 128, 2)
    got, info = run_sddmm_plan(gpu_lib, w, Xr, w.X, 8, feat_hint=128)
    assert info["n_runs"] >= w.nnz // 512
    assert np.array_equal(got, run_sddmm(gpu_lib, w, Xr, w.X))


def test_sddmm_plan_slices_that_find_no_memory_are_left_out(gpu_lib):
    """An allocation that only column slices ask for may fail: the plan then lists all rows.  (A caller's allocator that refuses
    one size, an error code and no GPU work.)"""
    from paper_2207_04606_amd import binding
    w = matrix_with_long_rows(900, 600, 3001, 5, 128)
    Xr = left_operand(w, 128, 1)
    want = run_sddmm(gpu_lib, w, Xr, w.X)
    asked, refuse = [], set()

    @binding._ALLOC_FN
    def take(nbytes, ctx, stream):
        asked.append(int(nbytes))
        return None if int(nbytes) in refuse else binding._torch_alloc(nbytes, ctx, stream)

    assert gpu_lib.load_library().sptir_set_allocator(take, binding._torch_free, None) == 0
    try:
        for c in (1, 8):
            run_sddmm_plan(gpu_lib, w, Xr, w.X, c, feat_hint=16)          # (no slices)
        without = set(asked)
        asked.clear()
        got, info = run_sddmm_plan(gpu_lib, w, Xr, w.X, 8, feat_hint=128)
        assert info["n_runs"] < 64 and np.array_equal(got, want)
        only = [size for size in asked[:9] if size not in without]        # (the slices' come first)
        assert len(only) >= 8
        before = len(binding._torch_blocks)
        for size in only:
            refuse = {size}
            for c in (1, 8):
                got, info = run_sddmm_plan(gpu_lib, w, Xr, w.X, c, feat_hint=128)
                assert np.array_equal(got, want), size
                assert info["n_runs"] == 0 if c == 1 else info["n_runs"] >= w.nnz // 512, size
            assert len(binding._torch_blocks) == before
    finally:
        gpu_lib.sptir_set_allocator(False)
