"""Classes, row pointer and lists of matrices that fit one tile of 4096 rows (a single launch) and of those just beyond (two)."""
import numpy as np
import pytest

from paper_2404_04541_amd import workloads as W
from helpers import gpu_product, assert_matches_oracle

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("rows", [1, 63, 64, 257, 4095, 4096, 4097])
@pytest.mark.parametrize("force", [0, 1, 4])
def test_rows_of_every_class(rows, force):
    rng = np.random.default_rng(rows + force)
    d = np.array([0, 2, 12, 70, 160, 600])[rng.integers(0, 6, rows)]
    d[-1] = 12   # (the total is read from the last row's end)
    rp = np.concatenate([[0], np.cumsum(d)])
    A = W.CSR(rows, 700, rp, np.concatenate([np.sort(rng.choice(700, n, replace=False)) for n in d]).astype(np.int32), rng.standard_normal(int(rp[-1])))
    B = W.random_csr(700, 900, 8, 5)
    assert_matches_oracle(A, B, gpu_product(A, B, force), what=f"{rows} rows, force {force}")
