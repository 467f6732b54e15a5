"""The row count where its rounds of 4096 entries can go wrong: rows that end on a round's edge, cross one or several, hold one
entry less or more; empty rows between; rows of B of 2^19 entries or more, whose sums it does not keep in 32 bits."""
import numpy as np
import pytest

from paper_2404_04541_amd import binding as sg, workloads as W

pytestmark = pytest.mark.gpu


def count(a_lens, b_lens, seed):
    rng = np.random.default_rng(seed)
    k = len(b_lens)
    b_rp = np.concatenate([[0], np.cumsum(b_lens)]).astype(np.int64)
    b_col = np.concatenate([np.arange(n) for n in b_lens]).astype(np.int32)
    a_rp = np.concatenate([[0], np.cumsum(a_lens)]).astype(np.int64)
    a_col = rng.integers(0, k, int(a_rp[-1])).astype(np.int32)
    A = W.CSR(len(a_lens), k, a_rp, a_col, np.ones(a_col.size, np.float32))
    B = W.CSR(k, max(int(max(b_lens)), 1), b_rp, b_col, np.ones(b_col.size, np.float32))
    _, _, plan = sg.spgemm_symbolic(sg.Handle(), sg.to_device(A), sg.to_device(B))
    st = plan.stats()
    plan.destroy()
    products = np.asarray(b_lens, np.int64)[a_col]
    ip = np.add.reduceat(np.append(products, 0), np.minimum(a_rp[:-1], products.size)) * (np.asarray(a_lens) > 0)
    assert st["ip_total"] == int(ip.sum())
    edges = [0, 32, 128, 768, 1536, 65536, 1 << 20, 1 << 62]
    assert st["sym_bin_rows"][:7] == [int(((ip > lo) & (ip <= hi)).sum()) for lo, hi in zip(edges, edges[1:])]


@pytest.mark.parametrize("a_lens", [
    [4096], [4095, 1, 4096], [4097, 0, 0, 4095], [1, 4094, 1, 1], [20000, 3, 0, 12288, 1], [1] * 5000, [0] * 70 + [9000] + [0] * 70 + [2] * 3000,
])
def test_rows_at_the_edges_of_a_round(a_lens):
    count(a_lens, [1, 0, 3, 17, 5, 40], 3)


@pytest.mark.parametrize("longest", [(1 << 19) - 1, 1 << 19, (1 << 19) + 1])
def test_huge_rows_of_b(longest):
    count([1, 2, 0, 7, 100], [longest, 3, 0, 9], 4)


@pytest.mark.parametrize("a_lens", [[1024], [1025], [1023, 1, 0, 1], [1, 1022, 1], [0] * 63 + [1024], [17] * 60, [16] * 64, [16] * 63 + [17], [2] * 5000, [0, 0, 1]])
def test_chunks_of_about_as_many_entries_as_threads(a_lens):
    """Up to 1024 entries in a chunk of rows an entry is one thread's; with one more they are taken in rounds."""
    count(a_lens, [1, 0, 3, 17, 5, 40, 300], 5)


@pytest.mark.parametrize("entries", [900, 3000, 9000])
@pytest.mark.parametrize("longest", [(1 << 19) - 1, 1 << 19])
def test_a_huge_row_of_b_among_short_ones(longest, entries):
    """(the first, the only and a later round of a row hold it)"""
    count([entries, 5], [longest] + [1] * 3000, 6)


@pytest.mark.parametrize("rows", [65_535, 65_536, 70_001])
def test_count_where_a_stretch_of_rows_is_heavy(rows):
    """Rows of 6 entries, and 300 of 700 in a row: finer chunks from 65536 rows on."""
    a_lens = np.full(rows, 6)
    a_lens[31_000:31_300] = 700
    count(a_lens, [7] * 900, 8)
