"""Wide tiles of the dense workspace: rows of as many A entries as a workgroup describes at a time or keeps in registers (1024, 2048, and
one more of each), B in order and not, with and without block table and structure list; where the rule for them changes."""
import numpy as np
import pytest

from paper_2404_04541_amd import binding as sg, workloads as W
from helpers import gpu_product, assert_matches_oracle

pytestmark = pytest.mark.gpu


def operand(lens, cols, seed, dtype, ordered=True):
    """Rows of so many distinct columns, spread over the matrix."""
    rng = np.random.default_rng(seed)
    rows = [(np.arange(n, dtype=np.int64) * cols // n + rng.integers(0, max(1, cols // n))) % cols for n in lens]
    rows = [np.sort(r) if ordered else rng.permutation(r) for r in rows]
    rowptr = np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)
    return W.CSR(len(lens), cols, rowptr, np.concatenate(rows).astype(np.int32), W.draw_values(int(rowptr[-1]), -1.0, 1.0, dtype, seed, 1))


@pytest.mark.parametrize("dtype", [np.float64, np.float32])
@pytest.mark.parametrize("ordered", [True, False])
@pytest.mark.parametrize("cols", [20_000, 150_001, (1 << 20) + 5])
def test_entries_of_a_row(cols, ordered, dtype):
    A = operand([1023, 1024, 1025, 2047, 2048, 2049, 3100], 3200, 1, dtype)
    B = operand([20] * 3200, cols, 2, dtype, ordered)
    ref = None
    for options in ({}, {sg.OPT_COLUMN_LIST: 0}, {sg.OPT_BLOCK_TABLE: 0}, {sg.OPT_DIRECT_MIN: 256}, {sg.OPT_SEARCH_RATIO: 1000}, {sg.OPT_COLUMN_LIST: 100_000}):
        got = gpu_product(A, B, options=options)
        ref = assert_matches_oracle(A, B, got, ref=ref, what=f"{cols} columns, ordered {ordered}, {options}")
        assert got[3]["num_bin_rows"][5] + got[3]["num_bin_rows"][6] == A.rows


@pytest.mark.parametrize("cols, b_row, a_row, wide", [
    (1 << 19, 1000, 24, False), ((1 << 19) + 1, 1000, 24, True),   # 24 000 products a row, a thousand for an entry of A
    (150_000, 60, 400, True), (150_000, 600, 40, False),           # few products of an entry in a tile, many
    (800_000, 60, 90, False),                                      # 5400 products a row: searched tiles
])
def test_where_the_rule_changes(cols, b_row, a_row, wide):
    A = operand([a_row] * 40, 2000, 3, np.float32)
    B = operand([b_row] * 2000, cols, 4, np.float32)
    got = gpu_product(A, B, options={sg.OPT_SEARCH_RATIO: 4 if cols == 800_000 else 0})
    ref = assert_matches_oracle(A, B, got, what=f"{cols} columns")
    blocks = -(-cols // 8192)
    flags, sums = blocks * 2048 * A.rows, int(ref.cnt.sum()) * 8
    if cols == 800_000:
        assert got[3]["dense_search_tiles"] == A.rows == got[3]["dense_tiles"]
    else:   # (tiles are filled to the block)
        budget = (135 if wide else 66) * 1024
        assert (flags + sums) / budget <= got[3]["dense_tiles"] <= 1.5 * (flags + sums) / budget + A.rows


def test_an_unordered_row_of_many_entries_is_one_searched_tile():
    A = operand([150] * 20, 2000, 5, np.float64)
    B = operand([60] * 2000, 1_000_000, 6, np.float64, ordered=False)
    got = gpu_product(A, B)
    ref = assert_matches_oracle(A, B, got, what="unordered")
    assert 5632 < int(ref.cnt.min()) and int(ref.cnt.max()) <= 11264
    assert got[3]["dense_tiles"] == got[3]["dense_search_tiles"] == A.rows
