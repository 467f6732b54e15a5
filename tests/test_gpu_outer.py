"""GPU parity of the outer-product route (k -> i -> j through the accumulation / all arrays) against the
CPU checker's outer-product route and its row-wise route; the doubly compressed conversions against the
checker's builders."""
import numpy as np
import pytest

import oracle
from oracle import outer
from paper_2404_04541_amd import workloads as W
from helpers import RTOL

pytestmark = pytest.mark.gpu


def run_outer(A, B, capacity=0, handle=None):
    import torch
    from paper_2404_04541_amd import binding as sg
    h = handle or sg.Handle()
    dA, dB = sg.to_device(A), sg.to_device(B)
    Ac = sg.dcsc_from_csr(h, dA)
    Br = sg.dcsr_from_csr(h, dB)
    C = sg.spgemm_outer(h, Ac, Br, capacity)
    torch.cuda.synchronize()
    return Ac, Br, C


def check_against_oracles(A, B, C, what):
    ref = oracle.spgemm(A, B)
    assert np.array_equal(C.rowptr.cpu().numpy(), ref.rowptr), f"{what}: rowptr differs"
    assert np.array_equal(C.colidx.cpu().numpy(), ref.colidx), f"{what}: colidx differs"
    want = ref.values.astype(A.values.dtype).astype(np.float64)
    err = np.abs(C.values.cpu().numpy().astype(np.float64) - want)
    assert np.all(err <= RTOL[np.dtype(A.values.dtype)] * ref.absum), f"{what}: values off"
    return ref


@pytest.mark.parametrize("seed", range(8))
def test_outer_route_small_every_capacity(seed):
    u = W.rand_unit(seed, 960, np.arange(4, dtype=np.uint64))
    m, k, n = (1 + int(v * 300) for v in u[:3])
    dtype = np.float32 if seed % 2 else np.float64
    A = W.random_csr(m, k, 1 + u[3] * 6, seed, 961, dtype=dtype, sort_rows=seed % 3 != 0, allow_duplicates=seed % 4 == 0)
    B = W.random_csr(k, n, 4, seed, 962, dtype=dtype, sort_rows=seed % 3 != 1, allow_duplicates=seed % 4 == 1)
    for cap in (0, 1, 37, 1000):
        Ac, Br, C = run_outer(A, B, cap)
        check_against_oracles(A, B, C, f"seed {seed} capacity {cap}")
    # the conversions against the checker's builders
    cols, ptr, rows, vals = outer.dcsc_from_csr(A)
    assert np.array_equal(Ac.vec.cpu().numpy(), cols) and np.array_equal(Ac.ptr.cpu().numpy(), ptr)
    assert np.array_equal(Ac.idx.cpu().numpy(), rows) and np.array_equal(Ac.values.cpu().numpy(), vals)
    r, rp, c, v = outer.dcsr_from_csr(B)
    assert np.array_equal(Br.vec.cpu().numpy(), r) and np.array_equal(Br.ptr.cpu().numpy(), rp)
    assert np.array_equal(Br.idx.cpu().numpy(), c) and np.array_equal(Br.values.cpu().numpy(), v)
    # and the checker's own outer-product route gives the same structure
    orp, ocol, oval, oabs, _ = outer.spgemm_outer(A, B, 1000)
    assert np.array_equal(C.rowptr.cpu().numpy(), orp) and np.array_equal(C.colidx.cpu().numpy(), ocol)


def test_outer_route_empty_rows_columns_and_operands():
    from paper_2404_04541_amd import binding as sg
    h = sg.Handle()
    # most rows of A and most rows of B empty; columns of A that meet no row of B and the reverse
    A = W.random_csr(5000, 4000, 0.05, 31)
    B = W.random_csr(4000, 3000, 0.08, 32)
    _, _, C = run_outer(A, B, handle=h)
    ref = check_against_oracles(A, B, C, "hypersparse")
    assert int(ref.cnt.sum()) < 100
    Z = W.CSR(7, 5, np.zeros(8, np.int64), np.zeros(0, np.int32), np.zeros(0))
    Bn = W.random_csr(5, 6, 2, 0)
    for X, Y in ((Z, Bn), (W.random_csr(7, 5, 2, 1), W.CSR(5, 6, np.zeros(6, np.int64), np.zeros(0, np.int32), np.zeros(0)))):
        Ac, Br, C = run_outer(X, Y, handle=h)
        assert C.rowptr.cpu().tolist() == [0] * 8 and C.nnz == 0 and (Ac.vec.numel() == 0 or Br.vec.numel() == 0)
    with pytest.raises(sg.SpgemmError) as e:
        sg.spgemm_outer(h, sg.dcsc_from_csr(h, sg.to_device(Bn)), sg.dcsr_from_csr(h, sg.to_device(Bn)))   # 6 columns against 5 rows
    assert e.value.status == -2


def test_outer_route_config1_and_a_rectangular_case_with_several_batches():
    a, b = W.config1()
    _, _, C = run_outer(a, b)
    check_against_oracles(a, b, C, "config 1")
    a, b = W.config4(rows=200000, bcols=4096)     # 6.4e6 products, rectangular result; batches of 2^20
    _, _, C = run_outer(a, b, 1 << 20)
    check_against_oracles(a, b, C, "rectangular, 7 batches")
    a, b = W.config3(scale=12)                    # power-law: long runs of equal coordinates in a batch
    _, _, C = run_outer(a, b, 1 << 18)
    check_against_oracles(a, b, C, "power law")


@pytest.mark.parametrize("rows,n,per_a,per_b,capacity", [
    (300, 40, 9, 7, 2048),        # tiles of the merge that end between equal coordinates, many batches
    (300, 40, 9, 7, 2049),
    (300, 40, 9, 7, 4096),        # a tile of runs exactly, and one more
    (300, 40, 9, 7, 4097),
    (2, 3, 60, 3, 97),            # six coordinates, long runs
    (500, 70_000, 12, 40, 0),     # one batch of several ranges
    (60, 50_000, 400, 30, 50_000),  # a thousand products per column
])
def test_outer_tiles(rows, n, per_a, per_b, capacity):
    k = 3000 if rows > 400 else 700
    A = W.uniform_rows(rows, k, per_a, 51, 1, np.float64)
    B = W.uniform_rows(k, n, min(per_b, n), 51, 3, np.float64)
    _, _, C = run_outer(A, B, capacity)
    check_against_oracles(A, B, C, f"{rows} x {n}, capacity {capacity}")


def test_a_last_batch_that_is_cut_into_more_ranges_than_a_full_one():
    """A full batch of 1025 sort tiles goes in 513 ranges, the last one of 514 to 1024 tiles in a range per tile."""
    tile = 8192
    A = W.uniform_rows(2000, 2000, 64, 53, 1, np.float64)
    B = W.uniform_rows(2000, 3000, 128, 53, 3, np.float64)
    products = int(np.diff(B.rowptr)[A.colidx].sum())
    last = products % (1025 * tile)
    assert products // (1025 * tile) == 1 and 513 * tile < last <= 1024 * tile
    _, _, C = run_outer(A, B, 1025 * tile)
    check_against_oracles(A, B, C, "long last batch")


@pytest.mark.parametrize("batches_before", [1, 2])
def test_a_later_batch_that_no_bucket_holds(batches_before):
    """Batches of evenly spread products, then one that is all in one row: found out when the first batch has only been sorted (everything
    again, by passes alone), and when it has been merged (that batch again)."""
    rng = np.random.default_rng(61)
    m, n, per, batch = 200_000, 65_536, 40, 1_200_000
    spread = batches_before * batch // (per * 4)           # columns of A with four entries each
    late = batch // per                                    # columns with one entry, of row 7
    k = spread + late
    rows = np.concatenate([rng.integers(0, m, 4 * spread), np.full(late, 7)])
    cols = np.concatenate([np.repeat(np.arange(spread), 4), np.arange(spread, k)])
    key = np.unique(rows.astype(np.int64) * k + cols)
    rp = np.concatenate([[0], np.cumsum(np.bincount(key // k, minlength=m))]).astype(np.int64)
    A = W.CSR(m, k, rp, (key % k).astype(np.int32), rng.uniform(-1, 1, key.size))
    B = W.uniform_rows(k, n, per, 63, 3, np.float64)
    _, _, C = run_outer(A, B, batch)
    check_against_oracles(A, B, C, f"after {batches_before} batches")


@pytest.mark.parametrize("capacity", [50_000, 100_000, 1 << 20])
def test_batches_with_hardly_a_coordinate_of_their_own(capacity):
    """Every coordinate comes hundreds of times in every batch, and across their ends."""
    A = W.uniform_rows(40, 2000, 1000, 65, 1, np.float32)
    B = W.uniform_rows(2000, 30, 10, 65, 3, np.float32)
    _, _, C = run_outer(A, B, capacity)
    check_against_oracles(A, B, C, f"capacity {capacity}")


@pytest.mark.parametrize("dtype", [np.float64, np.float32])
def test_coordinates_repeated_in_either_array(dtype):
    """Two batches: every coordinate some times in the first and some times in the second, none among them, around the steps in which equal
    components are added up; the last coordinate's lie at the ends of both."""
    from paper_2404_04541_amd import binding as sg
    counts = [0, 1, 2, 3, 4, 5, 7, 8, 9, 11, 12, 13, 19, 20, 21, 600]
    pairs = [(x, y) for x in counts for y in counts][1:]
    first, second = np.array(pairs).T
    assert first.sum() == second.sum()
    K, most = 1200, 600
    cols = [np.concatenate([np.arange(x), most + np.arange(y)]) for x, y in pairs]
    rp = np.concatenate([[0], np.cumsum([c.size for c in cols])]).astype(np.int64)
    rng = np.random.default_rng(19)
    A = W.CSR(len(pairs), K, rp, np.concatenate(cols).astype(np.int32), rng.uniform(-1, 1, rp[-1]).astype(dtype))
    B = W.CSR(K, 1, np.arange(K + 1, dtype=np.int64), np.zeros(K, np.int32), rng.uniform(-1, 1, K).astype(dtype))
    _, _, C = run_outer(A, B, int(first.sum()))
    check_against_oracles(A, B, C, "repeats")
    got = C.values.cpu().numpy()
    for i, c in enumerate(cols):   # (added up in the order of the products, in double)
        s = np.float64(0)
        for v in A.values[rp[i]:rp[i + 1]].astype(np.float64) * B.values[c].astype(np.float64):
            s = s + v
        assert got[i] == dtype(s), pairs[i]
