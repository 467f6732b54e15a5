"""The classes of shorter rows in one launch: every pair of classes with and without dense rows, few rows and more than the launch is for,
columns that leave class 3 to its tile or to the hash workspace, rows without room in the plan, a plan that the caller keeps."""
import numpy as np
import pytest

from paper_2404_04541_amd import workloads as W
from helpers import gpu_product, assert_matches_oracle
from test_gpu_records import csr

pytestmark = pytest.mark.gpu
COLUMN_LIST = 4
LENGTHS = {0: 3, 1: 12, 2: 60, 3: 130, 5: 400}   # entries of a row of A (times 8 products) of each class


def operands(classes, each, cols, dtype, near=False, seed=3):
    rng = np.random.default_rng(seed)
    b = [np.sort(rng.choice(min(cols, 300) if near else cols, size=8, replace=False)) for _ in range(500)]
    a = [rng.choice(500, size=LENGTHS[c], replace=False) for _ in range(each) for c in classes]
    return csr(a, 500, dtype, seed), csr(b, cols, dtype, seed + 1)


@pytest.mark.parametrize("classes", [(0, 1), (0, 2), (1, 3), (2, 3), (0, 1, 2, 3), (0, 1, 2, 3, 5), (3, 5)])
@pytest.mark.parametrize("cols", [3000, 70000])
@pytest.mark.parametrize("limit", [1, 0, 8192])
def test_classes_in_one_launch(classes, cols, limit):
    A, B = operands(classes, 37, cols, np.float64)
    assert_matches_oracle(A, B, gpu_product(A, B, options={COLUMN_LIST: limit}), what=f"{classes} {cols} {limit}")


@pytest.mark.parametrize("dtype", [np.float64, np.float32])
@pytest.mark.parametrize("each", [1, 2000, 6000])
def test_few_and_many_rows(each, dtype):
    A, B = operands((0, 1, 2, 3), each, 5000, dtype, near=each == 2000)
    assert_matches_oracle(A, B, gpu_product(A, B), what=f"{each} rows of each class")


@pytest.mark.parametrize("dtype", [np.float64, np.float32])
@pytest.mark.parametrize("sym,num", [(True, True), (True, False), (False, False)])
def test_sides_of_the_limit(sym, num, dtype):
    """As many rows as share a launch in both phases, in the symbolic one alone (rows of class 2 come to class 3 in the numeric one) and in neither."""
    import torch
    limit = 16 * 4 * torch.cuda.get_device_properties(0).multi_processor_count   # workgroups: 16 times what the chip holds
    wgs = lambda rows: rows[0] // 16 + rows[1] // 4 + rows[2] // 4 + rows[3]  # noqa: E731
    each = {(True, True): limit / (1 / 16 + 1 / 4 + 2) - 8, (True, False): limit / (1 / 16 + 1 / 2 + 1) - 8, (False, False): limit / (1 / 16 + 1 / 2 + 1) + 16}[sym, num]
    A, B = operands((0, 1, 2, 3), int(each), 5000, dtype)
    got = gpu_product(A, B)
    assert (wgs(got[3]["sym_bin_rows"]) <= limit, wgs(got[3]["num_bin_rows"]) <= limit) == (sym, num)
    assert_matches_oracle(A, B, got, what=f"{int(each)} rows of each class")


@pytest.mark.parametrize("dense", [False, True])
def test_kept_plan_and_another_order(dense):
    import torch
    from paper_2404_04541_amd import binding as sg
    A, B = operands((0, 1, 2, 3, 5) if dense else (0, 1, 2), 2500, 40000, np.float64)
    h = sg.Handle()
    rp, _, plan = sg.spgemm_symbolic(h, sg.to_device(A), sg.to_device(B))
    for turned in (False, True):
        if turned:   # A's rows the other way round (B's, where rows are dense, may not change)
            for i in range(A.rows):
                lo, hi = A.rowptr[i], A.rowptr[i + 1]
                A.colidx[lo:hi] = A.colidx[lo:hi][::-1].copy()
        A.values[:] = W.draw_values(A.nnz, -1.0, 1.0, np.float64, 7 + turned, 1)
        col, val = sg.spgemm_numeric(h, plan, sg.to_device(A), sg.to_device(B), rp)
        torch.cuda.synchronize()
        assert_matches_oracle(A, B, (rp.cpu().numpy(), col.cpu().numpy(), val.cpu().numpy()), what=f"dense {dense} turned {turned}")
    plan.destroy()
