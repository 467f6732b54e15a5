"""The table of row lengths that the row count looks B's rows up in: the ends of its groups of 12 rows, rows that do not fit it (more than 255
entries), matrices on both sides of the rule, rows of A that begin where the row before begins, a column that is no row of B."""
import numpy as np
import pytest

from paper_2404_04541_amd import workloads as W
from helpers import gpu_product, assert_matches_oracle

pytestmark = pytest.mark.gpu


def operands(k, m, d, longest, near, seed=1):
    rng = np.random.default_rng(seed)
    rows = rng.integers(0, 4, k)
    rows[rng.integers(0, k, 5)] = longest
    rows[-1] = 3
    brp = np.concatenate([[0], np.cumsum(rows)])
    at = np.arange(brp[-1]) - np.repeat(brp[:-1], rows)
    B = W.CSR(k, 900, brp, (at * 3 + np.repeat(rng.integers(0, 100, k), rows)).astype(np.int32), rng.standard_normal(int(brp[-1])))
    cols = (np.arange(m)[:, None] * (k // m) + np.arange(d)) % k if near else np.sort(rng.integers(0, k // d, (m, d)) + np.arange(d) * (k // d), axis=1)
    cols[0, -1] = k - 1
    cols[1, 0] = 0
    A = W.CSR(m, k, np.arange(m + 1, dtype=np.int64) * d, cols.ravel().astype(np.int32), rng.standard_normal(m * d))
    return A, B


@pytest.mark.parametrize("k,m,d,longest,near", [
    (800004, 400000, 4, 40, False), (800005, 400000, 4, 255, False), (800015, 400000, 4, 256, False),   # (the last row of a group, the first, the longest that fit and do not)
    (786432, 400000, 4, 40, False), (786433, 400000, 4, 40, False), (800004, 266668, 7, 40, False), (800004, 266667, 7, 40, False),   # (sides of the rule)
    (800004, 400001, 4, 40, False), (800004, 400002, 4, 40, False), (800004, 400000, 4, 40, True)])
def test_products_are_counted_right(k, m, d, longest, near):
    A, B = operands(k, m, d, longest, near)
    assert_matches_oracle(A, B, gpu_product(A, B), what=f"{k} rows of B, {m} of A")


@pytest.mark.parametrize("column", [-1, 800004, 2147483647])
def test_a_column_that_is_no_row_is_refused(column):
    from paper_2404_04541_amd import binding as sg
    A, B = operands(800004, 400002, 4, 40, False)
    A.colidx[777777] = column
    with pytest.raises(sg.SpgemmError) as e:
        gpu_product(A, B)
    assert e.value.status == -8


def test_a_row_pointer_that_descends_is_refused():
    from paper_2404_04541_amd import binding as sg
    A, B = operands(800004, 400002, 4, 40, False)
    B.rowptr[345678] = B.rowptr[345680] + 5
    with pytest.raises(sg.SpgemmError) as e:
        gpu_product(A, B)
    assert e.value.status == -8
