"""The flag-list workspace of short rows: matrix widths at the edges of its flag words and at its limit, B rows of one to sixteen
entries (quads that are a lane's own, dealt, cut short), rows with more entries than lanes, repeated columns, any order, a kept plan."""
import numpy as np
import pytest

from paper_2404_04541_amd import binding as sg, workloads as W
from helpers import gpu_product, assert_matches_oracle

pytestmark = pytest.mark.gpu


def some_rows(lens, cols, rng, repeats, seed, dtype):
    rowptr = np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)
    colidx = np.concatenate([rng.integers(0, cols, n) if repeats else rng.permutation(cols)[:n] for n in lens] + [np.zeros(0)]).astype(np.int32)
    return W.CSR(len(lens), cols, rowptr, colidx, W.draw_values(int(rowptr[-1]), -1.0, 1.0, dtype, seed, 1))


@pytest.mark.parametrize("dtype", [np.float64, np.float32])
@pytest.mark.parametrize("cols", [1, 33, 2047, 2048, 2049, 4096, 4097, 8192, 8193])
def test_widths_row_lengths_and_orders(cols, dtype):
    rng = np.random.default_rng(cols)
    for repeats, b_most in ((True, 4), (False, 5), (True, 16), (False, 1)):
        b_lens = np.minimum(rng.integers(0, b_most + 1, 300), 1 << 30 if repeats else cols)
        a_lens = rng.integers(0, 1 + 128 // b_most, 500)       # at most 128 products a row: classes 0 and 1
        A = some_rows(a_lens, 300, rng, True, 7, dtype)
        B = some_rows(b_lens, cols, rng, repeats, 8, dtype)
        ref = None
        for force in (0, 1):                                   # 1: the sorted list
            got = gpu_product(A, B, force=force)
            ref = assert_matches_oracle(A, B, got, ref=ref, what=f"{cols} columns, rows of {b_most}, force {force}")
            assert got[3]["num_bin_rows"][0] > 0 and sum(got[3]["num_bin_rows"][2:7]) == 0


def test_numeric_phase_on_a_kept_plan_in_another_order():
    import torch
    rng = np.random.default_rng(3)
    A = some_rows(rng.integers(0, 12, 4000), 700, rng, False, 9, np.float64)
    B = some_rows(rng.integers(1, 11, 700), 900, rng, False, 10, np.float64)
    h = sg.Handle()
    dA, dB = sg.to_device(A), sg.to_device(B)
    rp, nnz, plan = sg.spgemm_symbolic(h, dA, dB)
    for turn in range(3):
        if turn:   # the entries of every row of B backwards
            for r in range(B.rows):
                s = slice(int(B.rowptr[r]), int(B.rowptr[r + 1]))
                B.colidx[s] = B.colidx[s][::-1].copy()
                B.values[s] = B.values[s][::-1] * 0.5
            dB = sg.to_device(B)
        col, val = sg.spgemm_numeric(h, plan, dA, dB, rp)
        torch.cuda.synchronize()
        assert_matches_oracle(A, B, (rp.cpu().numpy(), col.cpu().numpy(), val.cpu().numpy()), what=f"turn {turn}")
    plan.destroy()


@pytest.mark.parametrize("dtype", [np.float64, np.float32])
@pytest.mark.parametrize("cols", [1, 33, 2047, 2048, 2049, 4096, 4097, 8192, 8193])
@pytest.mark.parametrize("rows", [4095, 4096, 5003])
def test_enough_rows_for_the_flag_list(rows, cols, dtype):
    """Fewer than 4096 rows take the sorted list whatever the widths; no row of A is empty, so that all count."""
    rng = np.random.default_rng(rows + cols)
    for repeats, b_most in ((True, 4), (False, 5), (True, 16)):
        b_lens = np.minimum(rng.integers(1, 2 * b_most + 1, 300), 1 << 30 if repeats else cols)
        most = 128 // int(b_lens.max())
        A = some_rows(rng.integers(1, 1 + most, rows), 300, rng, True, 7, dtype)
        B = some_rows(b_lens, cols, rng, repeats, 8, dtype)
        got = gpu_product(A, B)
        assert_matches_oracle(A, B, got, what=f"{rows} rows, {cols} columns, rows of {b_most}")
        assert got[3]["num_bin_rows"][0] + got[3]["num_bin_rows"][1] == rows


def test_enough_rows_on_a_kept_plan_in_another_order():
    import torch
    rng = np.random.default_rng(4)
    A = some_rows(rng.integers(1, 12, 6000), 700, rng, False, 9, np.float64)
    B = some_rows(rng.integers(1, 11, 700), 900, rng, False, 10, np.float64)
    h = sg.Handle()
    dA, dB = sg.to_device(A), sg.to_device(B)
    rp, nnz, plan = sg.spgemm_symbolic(h, dA, dB)
    for turn in range(2):
        if turn:
            for r in range(B.rows):
                s = slice(int(B.rowptr[r]), int(B.rowptr[r + 1]))
                B.colidx[s] = B.colidx[s][::-1].copy()
                B.values[s] = B.values[s][::-1] * 0.5
            dB = sg.to_device(B)
        col, val = sg.spgemm_numeric(h, plan, dA, dB, rp)
        torch.cuda.synchronize()
        assert_matches_oracle(A, B, (rp.cpu().numpy(), col.cpu().numpy(), val.cpu().numpy()), what=f"turn {turn}")
    plan.destroy()
