"""Rows that are an earlier row of the same wave moved to other columns (discretised operators): many rows a wave, with rows between them
that differ in one column, in the length of one row of B, in their number of entries or in the order of these; results with more
columns than a record holds; matrices too wide for records; quads at the end of B's arrays; new values on a kept plan."""
import numpy as np
import pytest

from paper_2404_04541_amd import workloads as W
from helpers import gpu_product, assert_matches_oracle
from test_gpu_records import csr

pytestmark = pytest.mark.gpu


def operands(rows, cols, a_off, b_off, dtype, seed=5):
    """A: rows x rows and B: rows x cols, every row the same offsets from its number (wrapped around), with exceptions."""
    step = cols // rows
    b = []
    for k in range(rows):
        off = b_off[:-1] if k % 1013 == 0 else b_off
        b.append((k * step + np.asarray(off)) % cols)
    a = []
    for i in range(rows):
        r = (i + np.asarray(a_off)) % rows
        if i % 97 == 5: r[len(r) // 2] = (r[len(r) // 2] + 1) % rows      # one column differs
        elif i % 397 == 7: r = r[::-1].copy()                                  # another order
        elif i % 503 == 11: r = r[:-1]
        elif i % 1511 == 13: r = (i + np.arange(66)) % rows                    # more entries than lanes
        a.append(r)
    return csr(a, rows, dtype, seed), csr(b, cols, dtype, seed + 1)


# 13 x 13 products in few columns, the same in columns that hardly repeat (more than 192 of them), 60 entries, 2 long rows of B
SHAPES = {"near": (np.arange(13), np.arange(13)), "spread": (np.arange(13) * 20, np.arange(17)), "sixty": (np.arange(60), np.array([0, 1, 5])),
          "long": (np.array([0, 3]), np.arange(101))}


@pytest.mark.parametrize("dtype", [np.float64, np.float32])
@pytest.mark.parametrize("shape", sorted(SHAPES))
@pytest.mark.parametrize("cols", [20000, 20000 * 450])
def test_rows_moved(shape, cols, dtype):
    import torch
    from paper_2404_04541_amd import binding as sg
    A, B = operands(20000, cols, *SHAPES[shape], dtype)
    h = sg.Handle()
    dA, dB = sg.to_device(A), sg.to_device(B)
    rp, _, plan = sg.spgemm_symbolic(h, dA, dB)
    for seed in (1, 2):
        A.values[:] = W.draw_values(A.nnz, -1.0, 1.0, dtype, seed, 1)
        B.values[:] = W.draw_values(B.nnz, -1.0, 1.0, dtype, seed, 2)
        col, val = sg.spgemm_numeric(h, plan, sg.to_device(A), sg.to_device(B), rp)
        torch.cuda.synchronize()
        assert_matches_oracle(A, B, (rp.cpu().numpy(), col.cpu().numpy(), val.cpu().numpy()), what=f"{shape} {cols} values {seed}")
    plan.destroy()


@pytest.mark.parametrize("dtype", [np.float64, np.float32])
@pytest.mark.parametrize("last", [[0], [0, 1], [0, 3], [0, 4]])
@pytest.mark.parametrize("rows,alike,short", [(3000, True, 0), (3000, False, 0), (400, True, 40), (400, False, 40)])   # (short: rows of class 0 beside them, in one launch)
def test_a_first_entry_that_is_an_empty_row_at_the_end_of_b(rows, alike, short, last, dtype):
    rng = np.random.default_rng(rows + len(last))
    b = [(k % 100) + np.arange(5) for k in range(1000)] + [np.arange(n) for n in last]
    a = []
    for i in range(rows):
        r = (i + np.arange(40)) % 1000 if alike else rng.choice(1000, size=40, replace=False)
        a.append(np.concatenate([[1000], r]) if i % 5 == 2 or not alike else r)   # 200 products in 80 quads: 48 lanes of the second round have none
    a += [[1000, 3, 7]] * short
    A, B = csr(a, len(b), dtype, 3), csr(b, 150, dtype, 4)
    assert_matches_oracle(A, B, gpu_product(A, B), what=f"{rows} {alike} {last}")
