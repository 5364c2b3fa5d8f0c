"""Queues of the chunk lists that are cut (a row goes on in the next queue), in several launches of long rows.  The longest row a
chunk shorter than a queue, and an entry longer (dealt whole); cuts inside chunks and at their ends; every width of the lane groups."""
import numpy as np
import pytest
import torch

import oracle
import workloads
from gpu_helpers import upload
from test_gpu_parity import assert_y_close, say
from test_gpu_stream import Stream, decode

pytestmark = pytest.mark.gpu

QUEUE_KIND, ROW_BLOCK, BLOCKS = 3, 16, 40
# rows of a block; queues are 56 entries long where they have 408 or 409
LENGTHS = {"48 of 56": [48] + [40] * 9, "49 of 56": [49] + [40] * 9, "divides": [37] * 16, "spread": None}
CUT = ("48 of 56", "spread")


def rows_in_two_queues(sptir, hyb, info, w):
    """Rows with entries in more than one queue of a list (a partition a launch: a row has one piece in it).  Every queue begins
    with the first entries of a row, also of one that is cut, so that all queues begin at the partition's first columns."""
    st = Stream(sptir, hyb, info)
    ptr = sptir.sptir_hyb_array(hyb, "plan_rb_chunk_ptr")
    n_rb = info["n_row_blocks"]
    n = 0
    for b in range(n_rb * info["n_phases"]):
        queues, begun = {}, set()
        col0 = b // n_rb * info["part_width"]
        for k in range(int(ptr[b]), int(ptr[b + 1])):
            kind, _, real, col, row, _, _ = st.chunk(k)
            if kind == QUEUE_KIND:
                for s in np.flatnonzero(real):
                    queues.setdefault(int(row[s]), set()).add(s // 8)
                    if s // 8 not in begun:
                        begun.add(s // 8)
                        r = b % n_rb * info["row_block"] + int(row[s])
                        cols = w.indices[w.indptr[r]:w.indptr[r + 1]]
                        assert int(col[s]) + (col0 if st.compact else 0) == cols[cols >= col0][0]
        n += sum(len(q) > 1 for q in queues.values())
    return n


@pytest.mark.parametrize("wide", [0, 1])
@pytest.mark.parametrize("kind", sorted(LENGTHS))
@pytest.mark.parametrize("one_value", [False, True])
def test_cut_queues(gpu_lib, kind, wide, one_value):
    rng = np.random.default_rng(len(kind))
    deg = np.zeros(ROW_BLOCK * BLOCKS, dtype=np.int64)
    for b in range(BLOCKS):
        lens = LENGTHS[kind] or np.clip(rng.normal(37, 12, ROW_BLOCK).round(), 0, 64).astype(int)
        deg[ROW_BLOCK * b:ROW_BLOCK * b + len(lens)] = lens
    half = workloads.random_csr(deg.size, 350, deg, 3, 1)  # both partitions have rows of these lengths
    w = workloads.random_csr(deg.size, 700, 2 * deg, 3, 129)
    for r in range(deg.size):
        mine = half.indices[half.indptr[r]:half.indptr[r + 1]]
        w.indices[w.indptr[r]:w.indptr[r + 1]] = np.concatenate([mine, mine + 350])
        if one_value:
            w.values[w.indptr[r]:w.indptr[r + 1]] = w.values[w.indptr[r]] if deg[r] else 0
    d = upload(w)
    hyb = gpu_lib.sptir_hyb_build_ex(w.n_rows, 700, d.indptr, d.indices, d.values, 2, 6,
                                     {"rounds": 2, "parts_per_launch": 1, "row_block": ROW_BLOCK, "heavy_len": 1 << 20,
                                      "column_slices": 2, "wide_stream": wide})
    info = gpu_lib.sptir_hyb_info(hyb)
    assert info["n_heavy_pieces"] == 0 and info["n_phases"] == 2 and info["values_per_row"] == int(one_value)
    assert (rows_in_two_queues(gpu_lib, hyb, info, w) > 0) == (kind in CUT)
    rows, cols, vals = decode(gpu_lib, hyb, info, w)
    key = np.repeat(np.arange(w.n_rows, dtype=np.int64), np.diff(w.indptr)) * w.n_cols + w.indices
    o = np.argsort(rows * w.n_cols + cols, kind="stable")
    assert np.array_equal((rows * w.n_cols + cols)[o], key)
    assert np.array_equal(vals[o], w.values.view(np.int32).astype(np.int64))
    for feat in (1, 2, 3, 4, 16, 17, 32, 41, 64, 129):
        say(f"[cut queues] {kind} wide={wide} one_value={one_value} feat={feat}")
        X = np.ascontiguousarray(w.X[:, :feat])
        Yr, Sr = oracle.spmm_csr(w.n_rows, w.indptr, w.indices, w.values, X)
        Y = torch.full((w.n_rows, feat), float("nan"), device="cuda")
        gpu_lib.sptir_spmm(hyb, torch.from_numpy(X).cuda(), Y)
        assert_y_close(Y.cpu().numpy(), Yr, Sr, what=f"{kind} wide={wide} feat={feat}")
    hyb.destroy()
