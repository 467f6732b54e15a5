"""The walk over the pieces of B's rows in the dense workspaces: pieces around the sizes of quads and chunks, rows of
one length and of many, the ends of B's arrays, more pieces than are described at a time, and enough rows that their
runs are taken from both ends of the list."""
import numpy as np
import pytest

from paper_2404_04541_amd import workloads as W
from helpers import gpu_product, assert_matches_oracle

pytestmark = pytest.mark.gpu


def rows_of(lens, cols, rng, dtype, ordered=True):
    """A matrix whose rows have these many distinct columns."""
    col = [rng.choice(cols, n, replace=False, shuffle=not ordered) for n in lens]
    col = [np.sort(c) if ordered else c for c in col]
    rp = np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)
    c = np.concatenate(col).astype(np.int32)
    return W.CSR(len(lens), cols, rp, c, rng.uniform(-1, 1, c.size).astype(dtype))


def operands(lens, cols, products, dtype, rows=12, ordered=True, seed=5):
    """A's rows ask for rows of B of these lengths, in turn and the last row of B among them, until so many products are made."""
    rng = np.random.default_rng(seed)
    b_lens = np.asarray(list(lens) * (1200 // len(lens) + 1))[:1200]
    d = int(np.ceil(products / b_lens.mean()))
    a = [np.sort(np.append(rng.choice(1199, min(d, 1200) - 1, replace=False), 1199)) for _ in range(rows)]
    rp = np.arange(rows + 1, dtype=np.int64) * a[0].size
    c = np.concatenate(a).astype(np.int32)
    return W.CSR(rows, 1200, rp, c, rng.uniform(-1, 1, c.size).astype(dtype)), rows_of(b_lens, cols, rng, dtype, ordered)


@pytest.mark.parametrize("lens", [(2,), (3, 5), (4,), (15, 17), (16,), (31, 32, 33), (63, 64, 65), (64,), (127, 129), (255, 256, 257), (1, 1000), (1, 2, 3, 4, 60, 61, 700)])
@pytest.mark.parametrize("cols,dtype", [(3000, np.float32), (3000, np.float64), (300_000, np.float64), (600_000, np.float32)])
def test_pieces_around_the_sizes_of_chunks(lens, cols, dtype):
    A, B = operands(lens, cols, max(2100, 6 * max(lens)), dtype)
    got = gpu_product(A, B)
    assert_matches_oracle(A, B, got, what=f"pieces of {lens}")


@pytest.mark.parametrize("lens", [(2, 3), (7, 64, 65), (300,)])
@pytest.mark.parametrize("cols", [3000, 400_000, 1_200_000])
def test_pieces_of_unordered_rows(lens, cols):
    A, B = operands(lens, cols, 4000, np.float32, ordered=False)
    got = gpu_product(A, B)
    assert_matches_oracle(A, B, got, what=f"unordered pieces of {lens}")


@pytest.mark.parametrize("d", [1023, 1024, 1025, 3000])
def test_more_pieces_than_are_described_at_a_time(d):
    rng = np.random.default_rng(7)
    B = rows_of(rng.integers(1, 9, 4000), 20_000, rng, np.float64)
    a = [np.sort(rng.choice(4000, d, replace=False)) for _ in range(5)]
    A = W.CSR(5, 4000, np.arange(6, dtype=np.int64) * d, np.concatenate(a).astype(np.int32), rng.uniform(-1, 1, 5 * d))
    got = gpu_product(A, B)
    assert_matches_oracle(A, B, got, what=f"{d} pieces")


@pytest.mark.parametrize("rows", [32_767, 32_768, 32_771])
def test_runs_from_both_ends(rows):
    """64 runs for each of 512 workgroups; a hundredth of the rows is ten times as heavy."""
    rng = np.random.default_rng(9)
    B = rows_of(np.full(400, 200), 2500, rng, np.float32)
    d = np.where(np.arange(rows) % 100 == 7, 90, 9)
    c = np.concatenate([np.sort(rng.choice(400, n, replace=False)) for n in d]).astype(np.int32)
    A = W.CSR(rows, 400, np.concatenate([[0], np.cumsum(d)]).astype(np.int64), c, rng.uniform(-1, 1, c.size).astype(np.float32))
    got = gpu_product(A, B)
    assert_matches_oracle(A, B, got, what=f"{rows} rows")
    assert got[3]["sym_bin_rows"][4] == rows


@pytest.mark.parametrize("rows", [8191, 8192])
@pytest.mark.parametrize("cols", [2500, 262_144, 262_145])
def test_rows_for_smaller_workgroups(rows, cols):
    """Both sides of 32 rows for each of 256 compute units, and of 2^18 columns; rows of more A entries than 8 waves (512) and 16 (1024) describe at a time."""
    rng = np.random.default_rng(11)
    B = rows_of(rng.integers(100, 300, 300), cols, rng, np.float64)
    d = np.full(rows, 17)
    d[:10] = (511, 512, 513, 600, 1023, 1024, 1025, 1100, 1537, 2100)
    c = np.concatenate([np.sort(rng.choice(300, n, replace=n > 300)) for n in d]).astype(np.int32)   # (the long ones with repeats)
    A = W.CSR(rows, 300, np.concatenate([[0], np.cumsum(d)]).astype(np.int64), c, rng.uniform(-1, 1, c.size))
    got = gpu_product(A, B)
    assert_matches_oracle(A, B, got, what=f"{rows} rows of {cols} columns")
    assert sum(got[3]["sym_bin_rows"][4:7]) == rows


def test_tiles_of_changing_size():
    """Every other block of 8192 columns is nearly a tile by itself and the ones between hold an entry: as many tiles as the plan's bound allows for."""
    rng = np.random.default_rng(13)
    n = 400_000
    full = [np.sort(rng.choice(8192, 6100, replace=False)) + 16384 * b for b in range(n // 16384)]
    one = [np.array([16384 * b + 8192 + 5]) for b in range(n // 16384)]
    cols = np.sort(np.concatenate(full + one)).astype(np.int32)
    B = W.CSR(8, n, np.arange(9, dtype=np.int64) * cols.size, np.tile(cols, 8), rng.uniform(-1, 1, 8 * cols.size))
    rows = 700
    A = W.CSR(rows, 8, np.arange(rows + 1, dtype=np.int64), rng.integers(0, 8, rows).astype(np.int32), rng.uniform(-1, 1, rows))
    got = gpu_product(A, B)
    assert np.array_equal(got[0], np.arange(rows + 1, dtype=np.int64) * cols.size)
    assert np.array_equal(got[1], np.tile(cols, rows))
    want = A.values[:, None] * B.values.reshape(8, -1)[A.colidx]
    assert np.allclose(got[2].reshape(rows, -1), want, rtol=1e-15, atol=0)   # (one product an entry)


@pytest.mark.parametrize("rows,cols", [(16_383, 2500), (16_384, 2500), (8191, 1_200_000), (8195, 1_200_000)])
def test_wide_runs_from_both_ends(rows, cols):
    """64 runs for each of 256 workgroups: B's rows are unordered, which leaves the wide kernel; beyond 2^20 columns a row has a run for each span."""
    rng = np.random.default_rng(15)
    B = rows_of(np.full(300, 200), cols, rng, np.float32, ordered=False)
    d = np.where(np.arange(rows) % 100 == 7, 90, 9)
    c = np.concatenate([rng.choice(300, n, replace=False) for n in d]).astype(np.int32)
    A = W.CSR(rows, 300, np.concatenate([[0], np.cumsum(d)]).astype(np.int64), c, rng.uniform(-1, 1, c.size).astype(np.float32))
    got = gpu_product(A, B)
    assert_matches_oracle(A, B, got, what=f"{rows} rows of {cols} columns")
    assert got[3]["sym_bin_rows"][4] == rows and got[3]["dense_runs"] == rows * (2 if cols > 1 << 20 else 1)


def test_light_rows_have_a_place_in_a_short_list():
    """Many rows of a wide matrix, every fourth of which takes 73 KB of flag words; a list with room for two thirds of those alone."""
    from paper_2404_04541_amd import binding as sg
    rng = np.random.default_rng(17)
    rows, cols = 16_400, 600_000
    B = rows_of(np.full(400, 100), cols, rng, np.float32)
    d = np.where(np.arange(rows) % 4 == 1, 130, 30)
    c = np.concatenate([np.sort(rng.choice(400, n, replace=False)) for n in d]).astype(np.int32)
    A = W.CSR(rows, 400, np.concatenate([[0], np.cumsum(d)]).astype(np.int64), c, rng.uniform(-1, 1, c.size).astype(np.float32))
    want = gpu_product(A, B)
    assert want[3]["dense_search_tiles"] == int((d == 30).sum())
    got = gpu_product(A, B, options={sg.OPT_COLUMN_LIST: 200_000_000})
    assert got[3]["dense_search_tiles"] > rows // 8
    assert all(np.array_equal(got[i], want[i]) for i in (0, 1))
    assert np.allclose(got[2], want[2], rtol=1e-5, atol=1e-5)
