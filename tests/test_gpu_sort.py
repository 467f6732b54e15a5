"""The radix sort and the scans behind the unfolding and the doubly compressed formats, at the edges of their tiles."""
import numpy as np
import pytest

from oracle import outer
from paper_2404_04541_amd import workloads as W

pytestmark = pytest.mark.gpu

TILE = 8192            # entries of a sort tile
RANGES = 1024          # ranges a pass is cut into at most


def coordinates(n, shape, seed):
    d = [W.rand_below(seed, 700 + t, np.arange(n, dtype=np.uint64), e).astype(np.int32) for t, e in enumerate(shape)]
    return W.COO3(shape, *d, W.draw_values(n, -1.0, 1.0, np.float64 if seed % 2 else np.float32, seed, 710))


@pytest.mark.parametrize("n,shape", [
    (1, (1, 1, 1)),                                # no key bits at all
    (TILE - 1, (3, 5, 7)),                         # few digits, long runs of equal keys: stable order
    (TILE, (700, 900, 300)),
    (TILE + 1, (65536, 2, 32768)),                 # 32 key bits: the last width of the narrow keys
    (3 * TILE + 17, (65536, 4, 32768)),            # 33 key bits
    (TILE * RANGES, (300, 200, 129)),              # a tile per range
    (TILE * RANGES + 5, (1024, 2048, 2047)),       # two tiles per range, the last range short
])
def test_unfolding_at_the_edges_of_the_sort(n, shape):
    import torch
    from paper_2404_04541_amd import binding as sg
    h = sg.Handle()
    for mode in ((3,) if n > TILE else (1, 2, 3)):
        x = coordinates(n, shape, n % 97)
        got = sg.sptensor_unfold(h, mode, shape, *[torch.from_numpy(v).cuda() for v in (x.i, x.j, x.k, x.values)])
        kept = [d for d in range(3) if d != mode - 1]
        c = [x.i, x.j, x.k]
        row = c[kept[0]].astype(np.int64) * shape[kept[1]] + c[kept[1]]
        order = np.argsort(row * shape[mode - 1] + c[mode - 1], kind="stable")
        rowptr = np.searchsorted(row[order], np.arange(shape[kept[0]] * shape[kept[1]] + 1))
        assert np.array_equal(got.rowptr.cpu().numpy(), rowptr)
        assert np.array_equal(got.colidx.cpu().numpy(), c[mode - 1][order])
        assert np.array_equal(got.values.cpu().numpy(), x.values[order])


SAMPLE = 128           # entries of which one is counted before buckets are made


def sampled(n):
    t = np.arange((n + SAMPLE - 1) // SAMPLE, dtype=np.uint64)
    return (t * SAMPLE + ((t * 2654435761 & 0xffffffff) >> 25)).astype(np.int64)


@pytest.mark.parametrize("dtype", [np.float32, np.float64])
@pytest.mark.parametrize("n,shape,crowd,seen", [
    (200_003, (301, 997, 703), 0, True),          # (too few entries, and bits, for buckets)
    (1_048_576, (2000, 2000, 2000), 0, True),     # the last size without buckets
    (1_048_577, (2000, 2000, 2000), 0, True),     # and the first with: two passes and some 130 entries
    (3_000_000, (2000, 2000, 2000), 0, True),     # buckets of one wave's registers of four
    (12_600_000, (2000, 2000, 2000), 0, True),    # of eight
    (3_000_000, (2000, 2000, 2000), 700, True),   # some buckets of one workgroup
    (3_000_000, (2000, 2000, 2000), 700, False),
    (3_000_000, (2000, 2000, 2000), 4000, True),  # and some that are too long: by passes alone
    (3_000_000, (2000, 2000, 2000), 4000, False),  # where the sample meets none of their entries: sorted again
    (3_000_000, (600, 700, 900), 4000, True),     # (too few bits)
])
def test_buckets_of_the_sort(n, shape, crowd, seen, dtype):
    import torch
    from paper_2404_04541_amd import binding as sg
    g = torch.Generator(device="cuda").manual_seed(n + crowd)
    c = [torch.randint(e, (n,), device="cuda", generator=g) for e in shape]
    if crowd:   # so many entries more in each of a few rows, in few columns: repeated coordinates, which stay in their order
        at = torch.randperm(n, device="cuda", generator=g)
        if not seen:
            free = torch.ones(n, dtype=torch.bool, device="cuda")
            free[torch.from_numpy(sampled(n)[sampled(n) < n]).cuda()] = False
            at = at[free[at]]
        at = at[:crowd * 5]
        c[0][at] = 5
        c[1][at] = torch.arange(crowd * 5, device="cuda") % 5 * (shape[1] // 6)
        c[2][at] = torch.randint(40, (crowd * 5,), device="cuda", generator=g)
    v = torch.rand(n, dtype=torch.float64, device="cuda", generator=g).to(torch.float32 if dtype == np.float32 else torch.float64)
    got = sg.sptensor_unfold(sg.Handle(), 3, shape, *[x.to(torch.int32) for x in c], v)
    row = c[0] * shape[1] + c[1]
    order = torch.sort(row * shape[2] + c[2], stable=True).indices
    assert torch.equal(got.colidx.long(), c[2][order]) and torch.equal(got.values, v[order])
    assert torch.equal(got.rowptr, torch.searchsorted(row[order], torch.arange(shape[0] * shape[1] + 1, device="cuda")))


def test_crowded_entries_are_sorted_once():
    """Unfolding of entries that crowd in a corner of the tensor: 2.8 times as long as of evenly spread ones when their buckets were found too
    long after the sort; 1.0 times by passes alone, which buckets beat by a third where they are not."""
    import time
    import torch
    from paper_2404_04541_amd import binding as sg
    n, h = 10_000_000, sg.Handle()
    g = torch.Generator(device="cuda").manual_seed(3)
    u = [torch.rand(n, dtype=torch.float64, device="cuda", generator=g) for _ in range(3)]
    v = torch.rand(n, dtype=torch.float64, device="cuda", generator=g)
    even, crowded = ([(t ** p * 2048).to(torch.int32) for t in u] for p in (1, 3))

    def best(x):
        times = []
        for _ in range(8):
            torch.cuda.synchronize()
            t0 = time.perf_counter()
            sg.sptensor_unfold(h, 3, (2048,) * 3, *x, v)
            torch.cuda.synchronize()
            times.append(time.perf_counter() - t0)
        return min(times)
    assert best(crowded) < 2 * best(even)


@pytest.mark.parametrize("hub,late", [(0, False), (250, False), (4000, False), (4000, True)])   # (late: only in the second batch, behind the sample)
def test_outer_product_with_a_crowded_row(hub, late):
    """One row of A with so many entries more, times rows of B in few columns: its products are one bucket, or too many for one."""
    from oracle import spgemm as reference
    from paper_2404_04541_amd import binding as sg
    rng = np.random.default_rng(hub)
    rows, k, cols = 60000, 10000, 1 << 20
    lens = np.full(rows, 6)
    colidx = [np.sort(rng.choice(k, size=n, replace=False)) for n in lens]
    if hub: colidx[777] = np.sort(rng.choice(4000, size=hub, replace=False)) + (6000 if late else 0)
    rowptr = np.concatenate([[0], np.cumsum([c.size for c in colidx])]).astype(np.int64)
    A = W.CSR(rows, k, rowptr, np.concatenate(colidx).astype(np.int32), W.draw_values(int(rowptr[-1]), -1.0, 1.0, np.float64, 1, 3))
    bcol = np.concatenate([np.sort(rng.choice(cols if not hub else 500, size=8, replace=False)) for _ in range(k)]).astype(np.int32)
    B = W.CSR(k, cols, np.arange(k + 1, dtype=np.int64) * 8, bcol, W.draw_values(8 * k, -1.0, 1.0, np.float64, 2, 3))
    h = sg.Handle()
    C = sg.spgemm_outer(h, sg.dcsc_from_csr(h, sg.to_device(A)), sg.dcsr_from_csr(h, sg.to_device(B)), 1_500_000)
    ref = reference(A, B)
    assert np.array_equal(C.rowptr.cpu().numpy(), ref.rowptr) and np.array_equal(C.colidx.cpu().numpy(), ref.colidx)
    assert np.all(np.abs(C.values.cpu().numpy() - ref.values) <= 1e-12 * ref.absum)


@pytest.mark.parametrize("rows", [1, 4095, 4096, 4097, 4096 * 4096 + 3])
def test_doubly_compressed_rows_at_the_edges_of_the_scan(rows):
    import torch
    from paper_2404_04541_amd import binding as sg
    h = sg.Handle()
    lens = (W.rand_below(5, 720, np.arange(rows, dtype=np.uint64), 3) // 2).astype(np.int64)
    lens[-1] = 1
    rowptr = np.zeros(rows + 1, dtype=np.int64)
    np.cumsum(lens, out=rowptr[1:])
    n = int(rowptr[-1])
    A = W.CSR(rows, 40, rowptr, W.rand_below(5, 721, np.arange(n, dtype=np.uint64), 40).astype(np.int32), W.draw_values(n, -1.0, 1.0, np.float64, 5, 722))
    d = sg.dcsr_from_csr(h, sg.to_device(A))
    keep = np.flatnonzero(lens)
    assert np.array_equal(d.vec.cpu().numpy(), keep)
    assert np.array_equal(d.ptr.cpu().numpy(), np.concatenate([rowptr[keep], [n]]))
    if rows < 5000:
        cols, ptr, ids, vals = outer.dcsc_from_csr(A)
        c = sg.dcsc_from_csr(h, sg.to_device(A))
        assert np.array_equal(c.vec.cpu().numpy(), cols) and np.array_equal(c.ptr.cpu().numpy(), ptr)
        assert np.array_equal(c.idx.cpu().numpy(), ids) and np.array_equal(c.values.cpu().numpy(), vals)
