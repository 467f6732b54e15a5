"""Row count, binning and row pointer at the sizes where their shape changes: chunks of 64, 256 and 1024 rows, a last chunk that
is cut short, more tiles of row counts than a workgroup adds up by itself, rows of many entries between short ones."""
import numpy as np
import pytest

from paper_2404_04541_amd import workloads as W
from helpers import gpu_product, assert_matches_oracle

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("rows", [1, 63, 64, 65, 4095, 4097, 131_071, 131_073, 524_287, 524_288 + 1025, 4096 * 4096 + 4097])
def test_sizes_of_the_row_count(rows):
    rng = np.random.default_rng(rows)
    k, cols = 700, 900
    lens = np.zeros(rows, dtype=np.int64)
    some = rng.integers(0, rows, size=min(rows, 3000))
    lens[some] = rng.integers(0, 6, size=some.size)
    lens[rng.integers(0, rows, size=5)] = [2000, 17, 300, 64, 65]
    lens[-1] = 3
    rowptr = np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)
    nnz = int(rowptr[-1])
    A = W.CSR(rows, k, rowptr, rng.integers(0, k, size=nnz).astype(np.int32), W.draw_values(nnz, -1.0, 1.0, np.float64, 3, 1))
    b_lens = rng.integers(0, 9, size=k)
    b_cols = [np.sort(rng.choice(cols, size=n, replace=False)) for n in b_lens]
    B = W.CSR(k, cols, np.concatenate([[0], np.cumsum(b_lens)]).astype(np.int64), np.concatenate(b_cols).astype(np.int32),
              W.draw_values(int(b_lens.sum()), -1.0, 1.0, np.float64, 4, 1))
    assert_matches_oracle(A, B, gpu_product(A, B), what=f"{rows} rows")


@pytest.mark.parametrize("rows,hub", [(524_288, 0), (524_288 + 1025, 0), (700_001, 0), (700_001, 3000), (524_287, 0)])
def test_many_even_rows_and_a_heavy_one(rows, hub):
    """Rows of 0 to 3 entries: chunks of 1024 rows from 524 288 rows on, unless one of them holds a row of many entries."""
    rng = np.random.default_rng(rows + hub)
    k, cols = 5000, 600
    lens = rng.integers(0, 4, size=rows)
    lens[rows // 2] = hub if hub else 2
    rowptr = np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)
    nnz = int(rowptr[-1])
    A = W.CSR(rows, k, rowptr, rng.integers(0, k, size=nnz).astype(np.int32), W.draw_values(nnz, -1.0, 1.0, np.float32, 3, 1))
    B = W.uniform_rows(k, cols, 2, 81, 1, np.float32)
    assert_matches_oracle(A, B, gpu_product(A, B), what=f"{rows} rows, hub of {hub}")
