"""The plan's list, tile and run slabs of the dense workspace: fewer rows than workgroups, about as many, several slabs per
workgroup, and rows whose runs do not fit a slab."""
import numpy as np
import pytest

from paper_2404_04541_amd import workloads as W
from helpers import gpu_product, assert_matches_oracle

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("rows,mean,cols,b_mean", [
    (1, 60, 50_000, 60),           # one workgroup
    (255, 60, 50_000, 60),
    (257, 60, 50_000, 60),         # two rows in one workgroup, slab of one record
    (5000, 50, 9_001, 50),         # two records a slab
    (3, 1500, 3_000_000, 700),     # three spans, several runs in each: more than a slab of one record
])
def test_dense_rows_and_slabs(rows, mean, cols, b_mean):
    # (lengths near the mean: every row is long enough for the dense workspace)
    k = 2000
    A = W.uniform_rows(rows, k, mean, 91, 1, np.float64)
    B = W.uniform_rows(k, cols, b_mean, 91, 3, np.float64)
    got = gpu_product(A, B)
    assert_matches_oracle(A, B, got, what=f"{rows} dense rows")
    st = got[3]
    assert st["num_bin_rows"][5] + st["num_bin_rows"][6] == rows and st["dense_runs"] >= rows


@pytest.mark.parametrize("rows", [1, 2, 40, 300])
def test_every_long_row_finds_room_in_the_list(rows):
    """Rows of about 3000 entries over a million columns with hardly a column twice: each becomes one searched tile, which needs
    its columns in the list."""
    A = W.uniform_rows(rows, 3000, 6, 93, 1, np.float32)
    B = W.uniform_rows(3000, 1_000_000, 500, 93, 3, np.float32)
    got = gpu_product(A, B)
    assert_matches_oracle(A, B, got, what=f"{rows} rows")
    assert got[3]["dense_search_tiles"] == rows


@pytest.mark.parametrize("rows", [1, 40, 300])
def test_list_bytes_used_are_those_of_the_rows(rows):
    """Rows of about 3000 entries over a million columns keep their columns, four bytes each in groups of four; a list of 4 KB
    has room for none of them."""
    A = W.uniform_rows(rows, 3000, 6, 93, 1, np.float32)
    B = W.uniform_rows(3000, 1_000_000, 500, 93, 3, np.float32)
    got = gpu_product(A, B)
    assert_matches_oracle(A, B, got, what=f"{rows} rows")
    assert got[3]["plan_list_used"] == int(((np.diff(got[0]) + 3) // 4 * 4).sum()) * 4 <= got[3]["plan_list_bytes"]
    got = gpu_product(A, B, options={4: 4096})   # (SPGEMM_OPT_COLUMN_LIST)
    assert_matches_oracle(A, B, got, what=f"{rows} rows, no room")
    assert got[3]["plan_list_used"] == 0 and got[3]["plan_list_bytes"] == 4096


@pytest.mark.parametrize("cols", [100_000, 300_000])
@pytest.mark.parametrize("room", [2.0, 1.0, 0.6])
def test_rows_of_one_length_that_draw_at_the_same_moment(cols, room):
    """Several rows for each of hundreds of workgroups, all of about the same length, so that slabs run out together; lists for all of them
    with the ends of the slabs, for the rows alone, for some: what is written stays within the list and no row gets another's place."""
    A = W.uniform_rows(6000, 3000, 50, 97, 1, np.float32)
    B = W.uniform_rows(3000, cols, 50, 97, 3, np.float32)
    got = gpu_product(A, B)
    ref = assert_matches_oracle(A, B, got, what="any list")
    need = int(((ref.cnt + 3) // 4 * 4).sum()) * 4
    got = gpu_product(A, B, options={4: int(need * room)})   # (SPGEMM_OPT_COLUMN_LIST)
    assert_matches_oracle(A, B, got, ref=ref, what=f"room for {room} of the rows")
    assert 0 < got[3]["plan_list_used"] <= got[3]["plan_list_bytes"] <= need * room


@pytest.mark.parametrize("rows,mean,b_mean,cols", [(6000, 50, 50, 100_000), (6000, 50, 50, 300_000), (700, 300, 20, 400_000), (3000, 12, 400, 1_000_000)])
def test_every_row_of_one_length_finds_room(rows, mean, b_mean, cols):
    """Hardly a column twice, several rows for each workgroup: the list of a plan without a limit has room for all columns."""
    A = W.uniform_rows(rows, 3000, mean, 97, 1, np.float32)
    B = W.uniform_rows(3000, cols, b_mean, 97, 3, np.float32)
    got = gpu_product(A, B)
    ref = assert_matches_oracle(A, B, got, what=f"{rows} rows")
    assert got[3]["num_bin_rows"][5] + got[3]["num_bin_rows"][6] == rows
    assert got[3]["plan_list_used"] == int(((ref.cnt + 3) // 4 * 4).sum()) * 4
