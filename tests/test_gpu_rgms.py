"""GPU parity tests of the relational gather-matmul-scatter operator: through the C ABI, against the fp64 oracle.
Criterion: |Y_gpu - Y_oracle| <= 1e-5 * sum |a x w| per element of Y (float32 products, float32 sums inside a (relation,
row) pair, float64 sums over pairs in any order), and exactly 0 where that sum is 0."""
import numpy as np
import pytest
import torch

import oracle
import workloads
from test_gpu_parity import say

pytestmark = pytest.mark.gpu
Y_TOL = 1e-5


def run_rgms(sptir, w, k=-1, workspace_d_out=0, repeat=1):
    dev = "cuda"
    ip = torch.from_numpy(w.indptr).to(dev)
    ix = torch.from_numpy(w.indices).to(dev)
    va = torch.from_numpy(w.values).to(dev)
    h = sptir.sptir_rgms_build(w.n_rel, w.n, w.n, ip, ix, va, k, workspace_d_out)
    info = sptir.sptir_rgms_info(h)
    X, W = torch.from_numpy(w.X).to(dev), torch.from_numpy(w.W).to(dev)
    outs = []
    for _ in range(repeat):
        Y = torch.full((w.n, w.W.shape[2]), float("nan"), device=dev)
        sptir.sptir_rgms(h, X, W, Y)
        outs.append(Y.cpu().numpy())
    h.destroy()
    return (outs[0] if repeat == 1 else outs), info


def assert_y_close(Y_gpu, Y_ref, S_ref, what):
    Y_gpu = Y_gpu.astype(np.float64)
    assert np.isfinite(Y_gpu).all(), f"{what}: non-finite output"
    zero = S_ref == 0
    assert (Y_gpu[zero] == 0).all(), what
    ratio = np.abs(Y_gpu - Y_ref)[~zero] / S_ref[~zero]
    worst = float(ratio.max()) if ratio.size else 0.0
    assert worst <= Y_TOL, f"{what}: max normalised error {worst:.3e}"
    return worst


@pytest.mark.parametrize("d_in,d_out", [(32, 32), (32, 64), (64, 32), (128, 96), (64, 128)])
@pytest.mark.parametrize("k", [-1, 0, 2, 5])
@pytest.mark.parametrize("workspace", [0, 64, 128])
def test_rgms_small_graphs(gpu_lib, d_in, d_out, k, workspace):
    """workspace 0: atomics only; 64: the workspace serves d_out <= 64 and the wider calls fall back to atomics."""
    say(f"[rgms] d_in={d_in} d_out={d_out} k={k} workspace={workspace}")
    w = workloads.make_hetero("hetero_tiny", seed=d_in + d_out + k, d_in=d_in, d_out=d_out)
    Y, info = run_rgms(gpu_lib, w, k, workspace)
    assert info["nnz"] == w.nnz and info["n_relations"] == w.n_rel and info["max_bucket_log2"] == (5 if k < 0 else k)
    assert info["workspace_d_out"] == workspace
    Yr, Sr = oracle.rgms(w.n_rel, w.n, w.indptr, w.indices, w.values, w.X, w.W)
    assert_y_close(Y, Yr, Sr, f"d_in={d_in} d_out={d_out} k={k}")


def test_rgms_long_rows_and_empty_relations(gpu_lib):
    """One (relation, row) pair with thousands of entries (several remainder tiles), relations without entries,
    rows without entries."""
    rng = np.random.default_rng(4)
    n, n_rel = 2500, 6
    trip = set()
    for j in rng.choice(n, 2300, replace=False):
        trip.add((1, 17, int(j)))                       # a very long stacked row
    for _ in range(4000):
        trip.add((int(rng.choice([0, 1, 4])), int(rng.integers(0, n // 2)), int(rng.integers(0, n))))   # 2, 3, 5 empty
    key = np.array(sorted((r * n + i) * n + j for r, i, j in trip), dtype=np.int64)
    stacked = key // n
    counts = np.bincount(stacked, minlength=n_rel * n)
    indptr = np.zeros(n_rel * n + 1, dtype=np.int64); np.cumsum(counts, out=indptr[1:])
    w = workloads.HeteroWorkload("long", n, n_rel, indptr.astype(np.int32), (key % n).astype(np.int32),
                                 rng.uniform(-1, 1, key.shape[0]).astype(np.float32),
                                 rng.standard_normal((n, 32)).astype(np.float32),
                                 rng.standard_normal((n_rel, 32, 32)).astype(np.float32))
    Yr, Sr = oracle.rgms(n_rel, n, w.indptr, w.indices, w.values, w.X, w.W)
    for workspace in (0, 32):
        Y, info = run_rgms(gpu_lib, w, workspace_d_out=workspace)
        assert_y_close(Y, Yr, Sr, f"long rows workspace={workspace}")


def test_rgms_reduces_to_spmm(gpu_lib):
    """One relation and W = I: the operator is Y = A X; 0/1 products are exact, so only the summation order differs."""
    w0 = workloads.make_config("small")
    n, feat = w0.n_rows, 32
    rng = np.random.default_rng(2)
    X = rng.standard_normal((n, feat)).astype(np.float32)
    w = workloads.HeteroWorkload("single", n, 1, w0.indptr, w0.indices, w0.values, X, np.eye(feat, dtype=np.float32)[None])
    Yr, Sr = oracle.spmm_csr(n, w0.indptr, w0.indices, w0.values, X)
    for workspace in (0, 32):
        Y, info = run_rgms(gpu_lib, w, workspace_d_out=workspace)
        assert_y_close(Y, Yr, Sr, f"single relation workspace={workspace}")


def test_rgms_edge_cases_and_errors(gpu_lib):
    dev = "cuda"
    # no entries at all: Y is still overwritten with zeros
    ip = torch.zeros(3 * 10 + 1, dtype=torch.int32, device=dev)
    ix = torch.zeros(0, dtype=torch.int32, device=dev); va = torch.zeros(0, device=dev)
    h = gpu_lib.sptir_rgms_build(3, 10, 10, ip, ix, va)
    Y = torch.full((10, 32), float("nan"), device=dev)
    gpu_lib.sptir_rgms(h, torch.zeros(10, 32, device=dev), torch.zeros(3, 32, 32, device=dev), Y)
    assert (Y == 0).all()
    with pytest.raises(gpu_lib.SptirError):        # feature sizes the matrix-core path does not cover
        gpu_lib.sptir_rgms(h, torch.zeros(10, 48, device=dev), torch.zeros(3, 48, 32, device=dev), Y)
    with pytest.raises(ValueError):
        gpu_lib.sptir_rgms(h, torch.zeros(10, 32, device=dev), torch.zeros(2, 32, 32, device=dev), Y)
    with pytest.raises(gpu_lib.SptirError):        # a bucket count beyond what the builder supports
        gpu_lib.sptir_rgms_build(7, 10, 10, torch.zeros(7 * 10 + 1, dtype=torch.int32, device=dev), ix, va, 9)
    with pytest.raises(gpu_lib.SptirError):        # workspace width not a multiple of 32
        gpu_lib.sptir_rgms_build(3, 10, 10, ip, ix, va, -1, 48)
    h.destroy()


def capped_hetero(seed, n, n_rel, cap, d=32):
    """A heterogeneous graph whose every (relation, row) pair has between 0 and `cap` entries."""
    rng = np.random.default_rng(seed)
    counts = rng.integers(0, cap + 1, n_rel * n)
    counts[rng.random(n_rel * n) < 0.5] = 0
    counts[rng.integers(0, n_rel * n, 8)] = cap          # the cap is reached
    indptr = np.zeros(n_rel * n + 1, dtype=np.int64); np.cumsum(counts, out=indptr[1:])
    indices = np.concatenate([np.sort(rng.choice(n, int(m), replace=False)) for m in counts if m] or [np.zeros(0)])
    return workloads.HeteroWorkload("capped", n, n_rel, indptr.astype(np.int32), indices.astype(np.int32),
                                    rng.uniform(-1, 1, indices.shape[0]).astype(np.float32),
                                    rng.standard_normal((n, d)).astype(np.float32),
                                    rng.standard_normal((n_rel, d, d)).astype(np.float32))


def test_rgms_workspace_path_is_reproducible(gpu_lib):
    """With the workspace every sum has a fixed order: calls agree bit for bit."""
    wl = capped_hetero(9, 700, 5, 32)
    assert np.diff(wl.indptr).max() == 32
    (Y1, Y2, Y3), info = run_rgms(gpu_lib, wl, workspace_d_out=32, repeat=3)
    assert info["max_bucket_log2"] == 5
    assert np.array_equal(Y1, Y2) and np.array_equal(Y1, Y3)
    Yr, Sr = oracle.rgms(wl.n_rel, wl.n, wl.indptr, wl.indices, wl.values, wl.X, wl.W)
    assert_y_close(Y1, Yr, Sr, "capped workspace")
    # and on a graph with longer pairs the two paths agree with the oracle to rounding
    w = workloads.make_hetero("hetero_a")
    assert np.diff(w.indptr).max() > 32
    Ya, _ = run_rgms(gpu_lib, w, workspace_d_out=0)
    Yb, _ = run_rgms(gpu_lib, w, workspace_d_out=32)
    Yr, Sr = oracle.rgms(w.n_rel, w.n, w.indptr, w.indices, w.values, w.X, w.W)
    assert_y_close(Ya, Yr, Sr, "atomics"); assert_y_close(Yb, Yr, Sr, "workspace")


@pytest.mark.parametrize("workspace", [0, 32])
@pytest.mark.parametrize("name", ["hetero_a", "hetero_b", "hetero_c", "hetero_d", "hetero_e"])
def test_rgms_named_configs(gpu_lib, name, workspace):
    w = workloads.make_hetero(name)
    Y, info = run_rgms(gpu_lib, w, workspace_d_out=workspace)
    say(f"[rgms config] {name}: nnz={w.nnz} pairs={info['n_stacked_rows_stored']} pads={info['n_pad_slots']} "
        f"tiles={info['n_tiles']}")
    Yr, Sr = oracle.rgms(w.n_rel, w.n, w.indptr, w.indices, w.values, w.X, w.W)
    worst = assert_y_close(Y, Yr, Sr, name)
    say(f"[rgms config] {name}: max_err={worst:.2e}")


@pytest.mark.parametrize("workspace", [0, 160])
@pytest.mark.parametrize("n,n_rel,d_in,d_out", [(1, 3, 32, 32), (31, 2, 32, 96), (257, 1, 64, 32), (700, 3, 32, 160),
                                                (4000, 2, 128, 64), (60_000, 4, 32, 32), (9000, 1, 128, 128)])
def test_rgms_tile_edges(gpu_lib, n, n_rel, d_in, d_out, workspace):
    """Pairs of 1, 4 +- 1, 8 +- 1, 64 +- 1 and 1500 entries (steps, pieces and batches of a tile), cells of 15 to 17 pairs,
    row blocks of several sizes, undivided, divided and shared between workgroups, one and several passes over Y."""
    check_tile_edges(gpu_lib, n, n_rel, d_in, d_out, workspace)


def check_tile_edges(gpu_lib, n, n_rel, d_in, d_out, workspace):
    rng = np.random.default_rng(n + d_out)
    counts = np.zeros(n_rel * n, dtype=np.int64)
    lens = np.minimum([1, 1, 2, 3, 4, 5, 7, 8, 9, 63, 64, 65], n)
    some = rng.choice(n_rel * n, min(n_rel * n, 3000), replace=False)
    counts[some] = rng.choice(lens, some.size)
    counts[: min(17, n_rel * n)] = 1
    counts[int(rng.integers(n_rel * n))] = min(1500, n)
    w0 = workloads.random_csr(n_rel * n, n, counts, 3, 1, "uniform")
    w = workloads.HeteroWorkload("edges", n, n_rel, w0.indptr, w0.indices, w0.values,
                                 rng.standard_normal((n, d_in)).astype(np.float32),
                                 rng.standard_normal((n_rel, d_in, d_out)).astype(np.float32))
    (Y, Y2), info = run_rgms(gpu_lib, w, workspace_d_out=workspace, repeat=2)
    assert info["n_stacked_rows_stored"] == int((counts > 0).sum()) and info["nnz"] == w.nnz
    Yr, Sr = oracle.rgms(n_rel, n, w.indptr, w.indices, w.values, w.X, w.W)
    assert_y_close(Y, Yr, Sr, f"n={n} d_in={d_in} d_out={d_out}")
    assert np.array_equal(Y, Y2) if workspace >= d_out else np.allclose(Y, Y2, rtol=1e-4, atol=1e-4)
    return info


def test_rgms_features_beyond_4_gb(gpu_lib):
    """Offsets into an X of more than 4 GB."""
    n_cols, d = (1 << 23) + 100, 128
    cols = [3, 1 << 22, (1 << 23) - 1, 1 << 23, n_cols - 1]
    ip = torch.tensor([0, 2, 5], dtype=torch.int32, device="cuda")
    ix = torch.tensor([cols[0], cols[3], cols[1], cols[2], cols[4]], dtype=torch.int32, device="cuda")
    va = torch.tensor([1.0, 2.0, -1.0, 0.5, 3.0], device="cuda")
    X = torch.zeros(n_cols, d, device="cuda")
    X[cols] = torch.randn(len(cols), d, device="cuda")
    W = torch.randn(1, d, 32, device="cuda")
    h = gpu_lib.sptir_rgms_build(1, 2, n_cols, ip, ix, va)
    Y = torch.full((2, 32), float("nan"), device="cuda")
    gpu_lib.sptir_rgms(h, X, W, Y)
    rows = X[ix.long()].cpu().double() * va.cpu().double()[:, None]
    want = torch.stack([rows[:2].sum(0), rows[2:].sum(0)]) @ W[0].cpu().double()
    assert torch.allclose(Y.cpu().double(), want, rtol=1e-4, atol=1e-3)
    h.destroy()


@pytest.mark.parametrize("workspace", [0, 128])
@pytest.mark.parametrize("n,n_rel,d_in,d_out", [(300, 5, 32, 32), (300, 5, 64, 64), (2000, 3, 128, 128), (9000, 2, 32, 64)])
def test_rgms_non_finite_rows_stay_with_their_rows(gpu_lib, n, n_rel, d_in, d_out, workspace):
    """A row of X with a NaN or an infinity reaches the rows of Y that have an entry naming it and no others, whatever
    tile, step of four or repeated last entry it shares with theirs; an infinite value of A and an infinite W[r]
    likewise.  (Which of infinity and NaN comes out depends on the order of the sums; that it is not finite does not.)"""
    rng = np.random.default_rng(n + d_in)
    check_non_finite_rows(gpu_lib, n, n_rel, d_in, d_out, workspace, np.minimum(rng.integers(0, 4, n_rel * n), n), rng)


def check_non_finite_rows(gpu_lib, n, n_rel, d_in, d_out, workspace, counts, rng):
    counts[rng.choice(n_rel * n, 40, replace=False)] = rng.choice([5, 8, 9, 16, 64, 65, 130], 40)  # several pieces, batches
    w = workloads.random_csr(n_rel * n, n, counts, 3, 1, "uniform")
    X = rng.standard_normal((n, d_in)).astype(np.float32)
    bad = rng.choice(n if counts.sum() > n else np.unique(w.indices), 6, replace=False)  # (columns that entries name)
    X[bad[0]] = np.nan
    X[bad[1], 0] = np.inf
    X[bad[2], d_in - 1] = -np.inf
    X[bad[3], d_in // 2] = np.nan
    X[n - 1, 3] = np.nan                             # the last column is the last entry of many a tile
    values = w.values.copy()
    values[rng.choice(values.size, 3, replace=False)] = [np.inf, -np.inf, np.nan]
    W = rng.standard_normal((n_rel, d_in, d_out)).astype(np.float32)
    for W_bad in (False, True):
        if W_bad:
            W[n_rel - 1, d_in // 3, 5] = np.inf
        hw = workloads.HeteroWorkload("non-finite", n, n_rel, w.indptr, w.indices, values, X, W)
        Y, info = run_rgms(gpu_lib, hw, workspace_d_out=workspace)
        with np.errstate(invalid="ignore", over="ignore"):
            Yr, Sr = oracle.rgms(n_rel, n, w.indptr, w.indices, values, X, W)
        finite = np.isfinite(Yr)
        assert finite.any() and not finite.all()
        wrong = np.isfinite(Y) != finite
        assert not wrong.any(), f"{int(wrong.sum())} of {int(finite.sum())} elements"
        assert_y_close(np.where(finite, Y, 0), np.where(finite, Yr, 0), np.where(finite, Sr, 0), "finite rows")
    return info


@pytest.mark.parametrize("d_in,d_out", [(32, 32), (64, 96), (128, 64)])
def test_rgms_blocks_of_512_rows(gpu_lib, d_in, d_out):
    """Many rows and few entries per relation: the largest row blocks, the last one with part of its rows."""
    say(f"[rgms 512] d_in={d_in} d_out={d_out}")
    assert check_tile_edges(gpu_lib, 512 * 512 + 77, 8, d_in, d_out, 0)["row_block"] == 512
    rng = np.random.default_rng(d_in)
    counts = (rng.random(8 * (512 * 512 + 1)) < 0.03).astype(np.int64)    # (16 entries a relation and block)
    assert check_non_finite_rows(gpu_lib, 512 * 512 + 1, 8, d_in, d_out, 0, counts, rng)["row_block"] == 512


@pytest.mark.parametrize("mean,rows", [(0.03, 512), (0.07, 512), (0.085, 256), (0.11, 256), (0.2, 256), (0.3, 128), (1.1, 32)])
def test_rgms_rows_of_a_block(gpu_lib, mean, rows):
    """So many that 32 entries are in a relation's part of a block, and 512 only where even those have fewer than 40."""
    n, n_rel = 512 * 512 + 5, 4
    counts = np.random.default_rng(1).poisson(mean, n_rel * n)
    w = workloads.random_csr(n_rel * n, n, counts, 1, 1)
    dev = lambda a: torch.from_numpy(a).cuda()
    h = gpu_lib.sptir_rgms_build(n_rel, n, n, dev(w.indptr), dev(w.indices), dev(w.values))
    assert gpu_lib.sptir_rgms_info(h)["row_block"] == rows
    h.destroy()
    if rows == 512:
        h = gpu_lib.sptir_rgms_build(n_rel, n, n, dev(w.indptr), dev(w.indices), dev(w.values), -1, 32)
        assert gpu_lib.sptir_rgms_info(h)["row_block"] == 256          # (tiles that take turns)
        h.destroy()


@pytest.mark.parametrize("workspace", [0, 96])
@pytest.mark.parametrize("d_in,d_out", [(32, 32), (32, 96), (64, 64), (128, 32)])
def test_rgms_quads_and_steps(gpu_lib, d_in, d_out, workspace):
    """Cells of 0 to 37 pairs of 0 to 5 entries each: pieces of up to four entries, quads and tiles of every length, places without
    an entry, with NaN in a row of X that a few pairs name and others share a step with, and with infinities where no sum has both signs: places
    without an entry multiply zeros, not a row of X, so an infinity stays one."""
    rng = np.random.default_rng(d_in + d_out)
    n, n_rel, block = 38 * 32, 3, 32                       # (32 rows per block: so many entries are in a cell)
    counts = np.zeros((n_rel, n), dtype=np.int64)
    for b in range(n // block):
        for r in range(n_rel):
            pairs = min(b, block)
            at = b * block + rng.choice(block, pairs, replace=False)
            counts[r, at] = [rng.integers(1, 6, pairs), np.full(pairs, 1 + b % 5), 1 + np.arange(pairs) % 4][r]
            if b > block:
                counts[r, at[: b - block]] += 4            # two pieces each
    w0 = workloads.random_csr(n_rel * n, n, counts.reshape(-1), 7, 1, "uniform")
    X = rng.standard_normal((n, d_in)).astype(np.float32)
    W = rng.standard_normal((n_rel, d_in, d_out)).astype(np.float32)
    for bad in (False, True):
        if bad:
            X[np.unique(w0.indices)[::97]] = np.nan
        w = workloads.HeteroWorkload("quads", n, n_rel, w0.indptr, w0.indices, w0.values, X, W)
        Y, info = run_rgms(gpu_lib, w, workspace_d_out=workspace)
        assert info["row_block"] == block and info["n_stacked_rows_stored"] == int((counts > 0).sum())
        with np.errstate(invalid="ignore"):
            Yr, Sr = oracle.rgms(n_rel, n, w.indptr, w.indices, w.values, X, W)
        finite = np.isfinite(Yr)
        assert finite.all() != bad and finite.any()
        assert np.array_equal(np.isfinite(Y), finite)
        assert_y_close(np.where(finite, Y, 0), np.where(finite, Yr, 0), np.where(finite, Sr, 0), f"d_in={d_in} d_out={d_out}")
    X = np.abs(np.nan_to_num(X)) + np.float32(0.1)
    X[np.unique(w0.indices)[::29], d_in // 2] = np.inf
    w = workloads.HeteroWorkload("infinities", n, n_rel, w0.indptr, w0.indices, w0.values, X, np.abs(W) + np.float32(0.1))
    Y, _ = run_rgms(gpu_lib, w, workspace_d_out=workspace)
    Yr, _ = oracle.rgms(n_rel, n, w.indptr, w.indices, w.values, w.X, w.W)
    assert (Yr == np.inf).any() and not np.isnan(Yr).any()
    assert np.array_equal(Y == np.inf, Yr == np.inf) and not np.isnan(Y).any()


@pytest.mark.parametrize("mean,rows", [(0.03, 256), (0.12, 256), (0.13, 128), (0.24, 128), (0.26, 64), (0.49, 64), (0.51, 32)])
def test_rgms_rows_of_a_block_with_a_workspace(gpu_lib, mean, rows):
    """Sixteen entries of a relation in a block are enough where tiles take turns."""
    n, n_rel = 512 * 128 + 5, 16
    counts = np.random.default_rng(1).poisson(mean, n_rel * n)
    w = workloads.random_csr(n_rel * n, n, counts, 1, 1)
    dev = lambda a: torch.from_numpy(a).cuda()
    h = gpu_lib.sptir_rgms_build(n_rel, n, n, dev(w.indptr), dev(w.indices), dev(w.values), -1, 32)
    assert gpu_lib.sptir_rgms_info(h)["row_block"] == rows
    h.destroy()


@pytest.mark.parametrize("blocks,mean,rows", [(160, 0.043, 512), (159, 0.043, 256), (160, 0.051, 256), (384, 0.051, 512), (383, 0.051, 256),
                                              (384, 0.085, 256)])
def test_rgms_fewer_blocks_of_512_rows(gpu_lib, blocks, mean, rows):
    """Blocks of 512 rows where 160 of them have fewer than 24 entries of a relation each, or 384 fewer than 40, and nobody shares their
    items (128 x 64 features: two workgroups an item of smaller blocks)."""
    say(f"[rgms 512, few] {blocks} blocks, {mean * 512:.0f} entries a relation and block")
    n, n_rel, d_in, d_out = 512 * blocks + 3, 5, 128, 64
    rng = np.random.default_rng(blocks)
    w = workloads.random_csr(n_rel * n, n, rng.poisson(mean, n_rel * n), 1, 1)
    X = rng.standard_normal((n, d_in)).astype(np.float32)
    W = rng.standard_normal((n_rel, d_in, d_out)).astype(np.float32)
    w = workloads.HeteroWorkload("few", n, n_rel, w.indptr, w.indices, w.values, X, W)
    Y, info = run_rgms(gpu_lib, w)
    assert info["row_block"] == rows
    Yr, Sr = oracle.rgms(n_rel, n, w.indptr, w.indices, w.values, w.X, w.W)
    assert_y_close(Y, Yr, Sr, f"{blocks} blocks")


@pytest.mark.parametrize("workspace", [0, 64])
@pytest.mark.parametrize("n,mean,rows", [(128 * 191, 0.4, 128), (128 * 192, 0.4, 96), (128 * 213 - 37, 0.4, 107), (128 * 254 + 1, 0.4, 128),
                                         (64 * 200 + 5, 0.9, 51), (256 * 230, 0.22, 230), (128 * 300 + 7, 0.4, (151, 128)),
                                         (64 * 400, 0.9, (50, 64)), (32 * 900 + 3, 1.5, (38, 32)), (128 * 800, 0.4, 128),
                                         (128 * 700 - 1, 0.4, (117, 128)), (64 * 1200 + 1, 0.9, (76, 64)), (64 * 1301, 0.9, 64)])
def test_rgms_whole_turns_of_blocks(gpu_lib, n, mean, rows, workspace):
    """Where blocks of a power of two rows are a few for every CU, there are as many as make whole turns of the CUs, of any number of rows
    (with a workspace, one turn); the last has part of its rows, or some have none."""
    rows = rows if isinstance(rows, int) else rows[workspace > 0]
    say(f"[rgms whole turns] {n} rows workspace={workspace}")
    if workspace:
        mean /= 2                                               # (16 entries of a relation fill a block's part)
    n_rel, d_in, d_out = 3, 64, 64
    rng = np.random.default_rng(n)
    w = workloads.random_csr(n_rel * n, n, rng.poisson(mean, n_rel * n), 1, 1)
    X = rng.standard_normal((n, d_in)).astype(np.float32)
    W = rng.standard_normal((n_rel, d_in, d_out)).astype(np.float32)
    w = workloads.HeteroWorkload("whole turns", n, n_rel, w.indptr, w.indices, w.values, X, W)
    (Y, again), info = run_rgms(gpu_lib, w, workspace_d_out=workspace, repeat=2)
    assert info["row_block"] == rows
    Yr, Sr = oracle.rgms(n_rel, n, w.indptr, w.indices, w.values, w.X, w.W)
    assert_y_close(Y, Yr, Sr, f"{n} rows")
    assert workspace == 0 or np.array_equal(Y, again)


@pytest.mark.parametrize("workspace", [0, 288])
@pytest.mark.parametrize("d_in,d_out", [(32, 32), (32, 256), (64, 288), (128, 160)])
def test_rgms_long_pairs(gpu_lib, d_in, d_out, workspace):
    """Pairs of 4 to 130 entries, whose pieces meet by fours and by twos before the product: as many of either in a cell as leave
    every remainder of the tiles of four and of eight, and rows of Y wider than a workgroup's."""
    say(f"[rgms long pairs] d_in={d_in} d_out={d_out} workspace={workspace}")
    rng = np.random.default_rng(d_in + d_out)
    n, n_rel, block = 38 * 32, 4, 32
    counts = np.zeros((n_rel, n), dtype=np.int64)
    for b in range(n // block):
        at = b * block + rng.permutation(block)
        pairs = min(b, block)
        counts[0, at[:pairs]] = 16                                   # fours only
        counts[1, at[:pairs]] = 8                                    # twos only
        counts[2, at] = rng.choice([0, 3, 4, 7, 8, 12, 13, 16, 17, 24, 28, 31, 33, 64, 130], block)
        counts[3, at[:1 + b % 5]] = [130, 15, 16, 48, 9][: 1 + b % 5]
    w0 = workloads.random_csr(n_rel * n, n, counts.reshape(-1), 11, 1, "uniform")
    X = rng.standard_normal((n, d_in)).astype(np.float32)
    W = rng.standard_normal((n_rel, d_in, d_out)).astype(np.float32)
    w = workloads.HeteroWorkload("long", n, n_rel, w0.indptr, w0.indices, w0.values, X, W)
    (Y, again), info = run_rgms(gpu_lib, w, workspace_d_out=workspace, repeat=2)
    assert info["row_block"] == block and info["n_stacked_rows_stored"] == int((counts > 0).sum())
    pieces = (counts.reshape(n_rel, n // block, block) + 3) // 4
    assert info["n_tiles"] == int(((pieces.sum(2) + 15) // 16).sum())
    Yr, Sr = oracle.rgms(n_rel, n, w.indptr, w.indices, w.values, X, W)
    assert_y_close(Y, Yr, Sr, f"d_in={d_in} d_out={d_out}")
    assert workspace == 0 or np.array_equal(Y, again)


@pytest.mark.parametrize("d_in,d_out,n_rel", [(128, 128, 32), (64, 128, 64), (128, 64, 40)])
def test_rgms_shared_items(gpu_lib, d_in, d_out, n_rel):
    """163 row blocks with a tile and more for every relation: an item's tiles read half a million elements of W and more, and four
    workgroups share it (128 x 64: none, or three).  The last block has part of its rows; rows without entries are 0."""
    say(f"[rgms shared items] d_in={d_in} d_out={d_out} n_rel={n_rel}")
    rng = np.random.default_rng(d_in + n_rel)
    n = 163 * 32 - 5
    counts = rng.choice([0, 0, 1, 2, 5], n_rel * n, p=[0.3, 0.2, 0.3, 0.15, 0.05]).reshape(n_rel, n)
    counts[:, ::37] = 0
    w0 = workloads.random_csr(n_rel * n, n, counts.reshape(-1), 13, 1, "uniform")
    w = workloads.HeteroWorkload("shared", n, n_rel, w0.indptr, w0.indices, w0.values,
                                 rng.standard_normal((n, d_in)).astype(np.float32),
                                 rng.standard_normal((n_rel, d_in, d_out)).astype(np.float32))
    (Y, Y2), info = run_rgms(gpu_lib, w, repeat=2)
    assert info["row_block"] == 32 and info["n_tiles"] * d_in * d_out >= 163 * 300_000
    Yr, Sr = oracle.rgms(n_rel, n, w.indptr, w.indices, w.values, w.X, w.W)
    assert_y_close(Y, Yr, Sr, f"d_in={d_in} d_out={d_out}")
    assert_y_close(Y2, Yr, Sr, f"d_in={d_in} d_out={d_out}, again")


def test_rgms_non_finite_rows_cost_nothing(gpu_lib):
    """A call on an X that is all NaN does what one on numbers does.  (1.0 times as long; sums formed a second time took 20 to 30.)"""
    rng = np.random.default_rng(5)
    n, n_rel = 40_000, 16
    w = workloads.random_csr(n_rel * n, n, rng.integers(0, 5, n_rel * n), 3, 1)
    dev = lambda a: torch.from_numpy(a).cuda()
    h = gpu_lib.sptir_rgms_build(n_rel, n, n, dev(w.indptr), dev(w.indices), dev(w.values))
    W = torch.ones(n_rel, 32, 32, device="cuda")
    Y = torch.empty(n, 32, device="cuda")

    def least_ms(X):
        best = float("inf")
        for _ in range(8):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            gpu_lib.sptir_rgms(h, X, W, Y)
            b.record()
            torch.cuda.synchronize()
            best = min(best, a.elapsed_time(b))
        return best

    finite = least_ms(torch.ones(n, 32, device="cuda"))
    nan = least_ms(torch.full((n, 32), float("nan"), device="cuda"))
    has_entries = np.diff(w.indptr).reshape(n_rel, n).sum(0) > 0
    assert np.array_equal(torch.isnan(Y).all(1).cpu().numpy(), has_entries)
    assert nan < 4 * finite, f"{nan:.3f} ms against {finite:.3f}"
    h.destroy()
