"""Rows of numeric class 3 (193 to 1536 entries): as tiles without structure up to 65536 columns (at most 1536 products), by their
tiles (more products), by the hash workspace (wider matrices, or on request); few and many entries of A, any order, repeats."""
import numpy as np
import pytest

from paper_2404_04541_amd import workloads as W
from helpers import gpu_product, assert_matches_oracle

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", [np.float64, np.float32])
@pytest.mark.parametrize("cols", [1537, 8192, 8193, 65536, 65537])
@pytest.mark.parametrize("ordered", [True, False])
def test_rows_of_class_3(cols, dtype, ordered):
    rng = np.random.default_rng(cols)
    k = 1300
    lens = np.concatenate([[1, 2, 255, 256, 257, 700, 1200], rng.integers(20, 120, 120)])
    a_cols = [rng.permutation(k)[:n] for n in lens]
    A = W.CSR(len(lens), k, np.concatenate([[0], np.cumsum(lens)]).astype(np.int64), np.concatenate(a_cols).astype(np.int32),
              W.draw_values(int(lens.sum()), -1.0, 1.0, dtype, 1, 1))
    for per in (1, 11, 24):   # products per entry of A; the columns of a row of B lie within a stretch of 1400 or less
        b = []
        for i in range(k):
            c = (int(rng.integers(0, 8)) + np.arange(per) * 50 + 13 * (i % 97)) % 1500
            if not ordered:
                c = rng.permutation(np.concatenate([c[: per // 2], c[: per - per // 2]]))
            b.append(np.sort(c) + (cols - 1500) if ordered else c + (cols - 1500))
        B = W.CSR(k, cols, np.arange(k + 1, dtype=np.int64) * per, np.concatenate(b).astype(np.int32),
                  W.draw_values(k * per, -1.0, 1.0, dtype, 2, 1))
        ref = None
        for force in (0, 2):   # 2: the hash workspace
            got = gpu_product(A, B, force=force)
            ref = assert_matches_oracle(A, B, got, ref=ref, what=f"{cols} columns, rows of {per}, force {force}")
        in_class = (ref.cnt > 192) & (ref.ip > 128)   # (no row reaches 1537 entries)
        assert got[3]["num_bin_rows"][3] == int(in_class.sum()) > 0
        if per == 11:
            assert bool(((ref.ip > 1536) & in_class).any()) and bool(((ref.ip <= 1536) & in_class).any())


@pytest.mark.parametrize("entries", [257, 300, 1025, 1100])
def test_rows_whose_last_entries_have_no_products(entries):
    """More entries of A than a workgroup describes at a time (256 in the tiles without structure, 1024 in the plan's tiles), those
    behind it with empty rows of B: the last round finds no piece, and the waves go on to count the columns all the same."""
    from paper_2404_04541_amd import binding as sg
    rng = np.random.default_rng(entries)
    full = 256 if entries < 1024 else 1024
    k = 1400
    b_lens = np.where(np.arange(k) < full, 4, 0)
    for cols in (3000, 70_000):
        B = W.CSR(k, cols, np.concatenate([[0], np.cumsum(b_lens)]).astype(np.int64),
                  np.concatenate([np.sort(rng.permutation(cols)[:n]) for n in b_lens]).astype(np.int32), W.draw_values(full * 4, -1.0, 1.0, np.float64, 5, 1))
        row = np.concatenate([np.arange(full), np.arange(full, entries)])
        rows = 600
        A = W.CSR(rows, k, np.arange(rows + 1, dtype=np.int64) * entries, np.tile(row, rows).astype(np.int32), W.draw_values(rows * entries, -1.0, 1.0, np.float64, 6, 1))
        for options in ({}, {sg.OPT_COLUMN_LIST: 0}):
            assert_matches_oracle(A, B, gpu_product(A, B, options=options), what=f"{cols} columns, {options}")


@pytest.mark.parametrize("dtype", [np.float64, np.float32])
def test_hashing_on_request_beside_dense_rows(dtype):
    """Hashing is asked for, and a dense row makes the tiles run: the rows of class 3 are still the hash workspace's, which their rows
    of B show by coming in another order than the plan's (the dense row's stay as they are)."""
    from test_gpu_records import csr, numeric_on_a_plan
    rng = np.random.default_rng(3)
    cols = 1 << 19
    used = np.sort(rng.choice(cols, size=1000, replace=False))
    b = [np.sort(rng.choice(used, size=8, replace=False)) for _ in range(900)] + [np.sort(rng.choice(cols, size=2000, replace=False)) for _ in range(3)]
    B = csr(b, cols, dtype, 4)
    A = csr([rng.choice(900, size=600, replace=False) for _ in range(60)] + [[900, 901, 902]], len(b), dtype, 5)
    B2 = W.CSR(B.rows, B.cols, B.rowptr, B.colidx.copy(), B.values.copy())
    for v in (B2.colidx, B2.values):
        v[:7200] = v[:7200].reshape(900, 8)[:, ::-1].ravel()
    st = numeric_on_a_plan((A, B), [(A, B), (A, B2)], "hashing", force=2)
    assert st["num_bin_rows"][3] == 60 and st["num_bin_rows"][5] + st["num_bin_rows"][6] == 1
