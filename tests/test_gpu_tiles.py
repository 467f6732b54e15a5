"""The dense workspace where its workgroups can go wrong: matrix widths on both sides of the change of geometry and of a block,
rows of as many A entries as a workgroup describes at a time (768 pieces, 1024 entries, and one more of each), with the block
table and the structure list and without."""
import numpy as np
import pytest

from paper_2404_04541_amd import binding as sg, workloads as W
from helpers import gpu_product, assert_matches_oracle

pytestmark = pytest.mark.gpu


def rows_of(lens, cols, seed, dtype):
    rowptr = np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)
    colidx = np.concatenate([np.arange(n, dtype=np.int64) * cols // n for n in lens]).astype(np.int32)
    return W.CSR(len(lens), cols, rowptr, colidx, W.draw_values(int(rowptr[-1]), -1.0, 1.0, dtype, seed, 1))


@pytest.mark.parametrize("dtype", [np.float64, np.float32])
@pytest.mark.parametrize("cols", [8191, 3 * 8192 + 5, (1 << 19) - 1, 1 << 19, (1 << 19) + 1])
def test_widths_and_entries_of_a_row(cols, dtype):
    A = rows_of([767, 768, 769, 1023, 1024, 1025, 2049], 2100, 95, dtype)
    B = W.uniform_rows(2100, cols, 7, 95, 3, dtype)
    for options in ({}, {sg.OPT_COLUMN_LIST: 0}, {sg.OPT_BLOCK_TABLE: 0}, {sg.OPT_DIRECT_MIN: 256}):
        got = gpu_product(A, B, force=3, options=options)
        ref = assert_matches_oracle(A, B, got, what=f"{cols} columns, {options}")
        assert got[3]["num_bin_rows"][5] == A.rows and int(ref.cnt.min()) > 1536


def test_some_rows_without_room_in_the_list():
    A = rows_of([300] * 40, 2100, 96, np.float64)
    B = W.uniform_rows(2100, 200_000, 40, 96, 3, np.float64)
    got = gpu_product(A, B, options={sg.OPT_COLUMN_LIST: 400_000})
    assert_matches_oracle(A, B, got, what="a short list")
    need = int(np.diff(got[0]).sum()) * 4
    assert 0 < got[3]["plan_list_used"] <= 400_000 < need
