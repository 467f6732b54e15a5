"""What the symbolic pass leaves of short rows for the numeric one: 64 and 65 entries in a row of A, 192 and 193
columns, quads that end at the end of B's arrays, lists too small for every row, too many columns for a record, new values on
a kept plan."""
import numpy as np
import pytest

from paper_2404_04541_amd import workloads as W
from helpers import gpu_product, assert_matches_oracle

pytestmark = pytest.mark.gpu
HASH, STAGED, COLUMN_LIST = 2, 4, 4


def csr(rows, cols, dtype, seed):
    lens = [len(r) for r in rows]
    rowptr = np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)
    colidx = np.concatenate([np.asarray(r, dtype=np.int32) for r in rows]) if sum(lens) else np.zeros(0, np.int32)
    return W.CSR(len(rows), cols, rowptr, colidx, W.draw_values(int(sum(lens)), -1.0, 1.0, dtype, seed, 1))


def operands(cols, dtype, seed=11):
    """Rows of 129 to 768 products: B rows of 1 to 13 entries, overlapping or not; the last rows of B end its arrays."""
    rng = np.random.default_rng(seed)
    b = [np.sort(rng.choice(min(cols, 400), size=1 + i % 13, replace=False)) for i in range(90)]           # few columns: much merging
    b += [np.sort(rng.choice(cols, size=1 + i % 13, replace=False)) for i in range(90)]                     # many columns
    b += [np.sort(rng.choice(cols, size=n, replace=False)) for n in (192, 193, 129, 768, 3, 2, 1, 1)]
    b += [np.arange(cols - 5, cols)]
    a = []
    for n in (20, 33, 63, 64, 65, 90):
        for lo in (0, 90):
            a.append(rng.choice(np.arange(lo, lo + 90), size=n, replace=False))
    a += [[180], [181], [182], [183], [180, 184], [180, 185, 186, 187], [182, 188], [], [182, 188, 188, 182]]
    a += [rng.choice(np.arange(0, 189), size=30, replace=False) for _ in range(40)]
    return csr(a, len(b), dtype, seed), csr(b, cols, dtype, seed + 1)


@pytest.mark.parametrize("dtype", [np.float64, np.float32])
@pytest.mark.parametrize("cols", [1000, 1 << 23, (1 << 23) + 1, 30_000_000])
@pytest.mark.parametrize("force", [0, HASH])
def test_recorded_rows(cols, dtype, force):
    A, B = operands(cols, dtype)
    assert_matches_oracle(A, B, gpu_product(A, B, force), what=f"cols={cols} force={force}")


@pytest.mark.parametrize("limit", [0, 4096, 16384])
def test_room_for_some_rows(limit):
    A, B = operands(5000, np.float64)
    assert_matches_oracle(A, B, gpu_product(A, B, options={COLUMN_LIST: limit}), what=f"list of {limit} bytes")


@pytest.mark.parametrize("force", [0, HASH])
def test_new_values_on_a_kept_plan(force):
    import torch
    from paper_2404_04541_amd import binding as sg
    A, B = operands(5000, np.float64)
    h = sg.Handle()
    h.set_option(sg.OPT_FORCE_WORKSPACE, force)
    dA, dB = sg.to_device(A), sg.to_device(B)
    rp, _, plan = sg.spgemm_symbolic(h, dA, dB)
    for seed in (21, 22):
        A.values[:] = W.draw_values(A.nnz, -1.0, 1.0, np.float64, seed, 1)
        B.values[:] = W.draw_values(B.nnz, -1.0, 1.0, np.float64, seed, 2)
        dA, dB = sg.to_device(A), sg.to_device(B)   # (other buffers as well)
        col, val = sg.spgemm_numeric(h, plan, dA, dB, rp)
        torch.cuda.synchronize()
        assert_matches_oracle(A, B, (rp.cpu().numpy(), col.cpu().numpy(), val.cpu().numpy()), what=f"values {seed}")
    plan.destroy()


@pytest.mark.parametrize("entries,long_rows", [((20,), 0), ((20,) * 9 + (21,), 0), ((14,), 0), ((14,), 1), ((14,), 2), ((14,) * 9 + (59,), 0), ((14,) * 4 + (59,), 0)])
@pytest.mark.parametrize("timing", [0, 1])
def test_slots_by_the_rows(entries, long_rows, timing):
    """Rows of 10 products an entry: 200 on average and a little more, one or two of 590 in 4200 (on both sides of one in 4096), many of them.  With the timing
    option the class has a launch of its own, without it shares one with a few shorter rows."""
    from paper_2404_04541_amd import binding as sg
    rng = np.random.default_rng(41)
    B = csr([np.sort(rng.choice(1500, 10, replace=False)) for _ in range(200)], 1500, np.float64, 42)
    rows = [rng.choice(200, entries[i % len(entries)], replace=False) for i in range(4200)]
    rows[1000:1000 + long_rows] = [rng.choice(200, 59, replace=False) for _ in range(long_rows)]
    rows[77:80] = [rng.choice(200, n, replace=False) for n in (1, 5, 9)]
    A = csr(rows, 200, np.float64, 43)
    got = gpu_product(A, B, options={sg.OPT_TIMING: timing})
    assert_matches_oracle(A, B, got, what=f"{entries}")
    assert got[3]["sym_bin_rows"][2] == 4197


def short_operands(b_rows, cols, dtype, sort_b, seed=31):
    """Rows of 0 to 128 products: one long B row, many short ones, more entries than lanes (most of them with empty B rows),
    columns hit several times; with more than 2^19 rows of B the row count describes the entries."""
    rng = np.random.default_rng(seed)
    used = 400
    b = []
    for i in range(used):
        n = [0, 1, 2, 3, 4, 5, 8, 16, 17, 31, 32, 33, 64, 127, 128][i % 15]
        pick = rng.choice(min(cols, 300) if i % 2 else cols, size=min(n, 300), replace=False)
        b.append(np.sort(pick) if sort_b else pick)
    lens = np.array([len(r) for r in b])
    a = []
    for total in list(range(0, 34)) + [63, 64, 65, 100, 127, 128]:
        for most in (4, 16, 128):
            row, left = [], total
            while left > 0:
                ok = np.flatnonzero((lens <= min(left, most)) & (lens > 0))
                k = int(rng.choice(ok))
                row.append(k)
                left -= int(lens[k])
            a.append(row)
            a.append(row[:len(row) // 2] + [0, 15, 30] * 30 + row[len(row) // 2:])   # (empty B rows between)
    B = csr(b, cols, dtype, seed)
    gap = max(0, b_rows - used)
    B = W.CSR(used + gap, cols, np.concatenate([B.rowptr, np.full(gap, B.rowptr[-1])]), B.colidx, B.values)
    return csr(a, used + gap, dtype, seed + 1), B


@pytest.mark.parametrize("dtype", [np.float64, np.float32])
@pytest.mark.parametrize("sort_b", [True, False])
@pytest.mark.parametrize("b_rows,cols", [(400, 300), (600_000, 300), (400, 1 << 23), (600_000, 1 << 25), (400, (1 << 25) + 1), (600_000, 40_000_000)])
def test_short_rows(b_rows, cols, dtype, sort_b):
    A, B = short_operands(b_rows, cols, dtype, sort_b)
    for options in ({}, {COLUMN_LIST: 0}, {COLUMN_LIST: 20_000}):   # (words for both bins, for none, for one)
        assert_matches_oracle(A, B, gpu_product(A, B, options=options), what=f"rows={b_rows} cols={cols} {options}")


@pytest.mark.parametrize("dtype", [np.float64, np.float32])
@pytest.mark.parametrize("force", [0, 1, HASH, 3, STAGED])
def test_rows_without_a_record_beside_rows_that_could_have_one(dtype, force):
    """200 rows of 500 products, ten of 10 000 products on 100 columns: short of entries for the hash workspace, too many products
    for a record and for the staged list."""
    import torch
    from paper_2404_04541_amd import binding as sg
    rng = np.random.default_rng(41)
    B = csr([np.sort(rng.choice(100, size=50, replace=False)) for _ in range(200)], 100, dtype, 42)
    A = csr([rng.choice(200, size=10, replace=False) for _ in range(200)] + [np.arange(200) for _ in range(10)], 200, dtype, 43)
    h = sg.Handle()
    h.set_option(sg.OPT_FORCE_WORKSPACE, force)
    dA, dB = sg.to_device(A), sg.to_device(B)
    rp, nnz, plan = sg.spgemm_symbolic(h, dA, dB)
    col = torch.full((nnz,), -1, dtype=torch.int32, device="cuda")
    val = torch.full((nnz,), float("nan"), dtype=dA.values.dtype, device="cuda")
    sg.spgemm_numeric(h, plan, dA, dB, rp, col, val)
    torch.cuda.synchronize()
    plan.destroy()
    assert_matches_oracle(A, B, (rp.cpu().numpy(), col.cpu().numpy(), val.cpu().numpy()), what=f"force {force}")


def reordered(M, rng):
    """The same entries, those of every row in another order (and in other buffers)."""
    at = np.concatenate([lo + rng.permutation(hi - lo) for lo, hi in zip(M.rowptr[:-1], M.rowptr[1:])] + [np.zeros(0, np.int64)])
    return W.CSR(M.rows, M.cols, M.rowptr.copy(), M.colidx[at], M.values[at])


def repeated(M, times):
    """The rows of M so many times over."""
    rowptr = np.concatenate([[0], np.cumsum(np.tile(np.diff(M.rowptr), times))]).astype(np.int64)
    return W.CSR(M.rows * times, M.cols, rowptr, np.tile(M.colidx, times), W.draw_values(M.nnz * times, -1.0, 1.0, M.values.dtype, 3, 1))


def numeric_on_a_plan(plan_of, calls, what, force=0, offset=0, options=None):
    """One plan for the operands plan_of, the numeric phase for each of calls in turn, every result compared.  Returns the plan's statistics."""
    import torch
    from paper_2404_04541_amd import binding as sg

    def device(M):   # offset: B's and A's columns and values do not start where their buffers do
        d = sg.to_device(M)
        for name in ("colidx", "values"):
            t = getattr(d, name)
            setattr(d, name, torch.cat([t.new_zeros(offset), t])[offset:])
        return d
    h = sg.Handle()
    h.set_option(sg.OPT_FORCE_WORKSPACE, force)
    for opt, value in (options or {}).items():
        h.set_option(opt, value)
    A, B = plan_of
    dA = device(A)
    dB = dA if B is A else device(B)
    rp, nnz, plan = sg.spgemm_symbolic(h, dA, dB)
    for n, (A, B) in enumerate(calls):
        dA = device(A)
        dB = dA if B is A else device(B)
        col = torch.full((nnz,), -1, dtype=torch.int32, device="cuda")
        val = torch.full((nnz,), float("nan"), dtype=dA.values.dtype, device="cuda")
        sg.spgemm_numeric(h, plan, dA, dB, rp, col, val)
        torch.cuda.synchronize()
        assert_matches_oracle(A, B, (rp.cpu().numpy(), col.cpu().numpy(), val.cpu().numpy()), what=f"{what}, call {n}")
    st = plan.stats()
    plan.destroy()
    return st


@pytest.mark.parametrize("dtype", [np.float64, np.float32])
@pytest.mark.parametrize("offset", [0, 1])
@pytest.mark.parametrize("kind", ["recorded", "small", "short", "described", "dense too"])
def test_entries_in_another_order_on_a_kept_plan(kind, dtype, offset):
    """The structure is the same whatever the order of a row's entries: a matrix that is assembled again may come in another one."""
    rng = np.random.default_rng(51)
    if kind == "recorded":
        A, B = operands(5000, dtype)
    elif kind == "dense too":   # (every class of rows; an ascending B has to stay so where rows are dense, so this one is not)
        A, B = W.random_csr(600, 500, 40, 52, dtype=dtype), W.random_csr(500, 4000, 30, 53, dtype=dtype, sort_rows=False)
    else:
        A, B = short_operands(600_000 if kind == "described" else 400, 3000, dtype, True)
        if kind != "small":   # (a plan that its caller holds has sorted words for short rows of a million products and more)
            A = repeated(A, 180)
            assert int(np.diff(B.rowptr)[A.colidx].sum()) > 1 << 20
    A2, B2 = reordered(A, rng), reordered(B, rng)
    numeric_on_a_plan((A, B), [(A2, B), (A, B2), (A, B), (A2, B2), (A, B)], kind, offset=offset)


def test_two_entries_exchanged_on_a_kept_plan():
    """The smallest change of order, at the first and last entries of the arrays; then an operand that is both A and B."""
    A, B = operands(5000, np.float64)
    calls = []
    for M, at in ((A, 0), (A, A.nnz - 2), (B, 1), (B, B.nnz - 2)):
        N = W.CSR(M.rows, M.cols, M.rowptr, M.colidx.copy(), M.values.copy())
        for v in (N.colidx, N.values):
            v[[at, at + 1]] = v[[at + 1, at]]
        row = int(np.searchsorted(M.rowptr, at, side="right")) - 1
        assert at + 1 < M.rowptr[row + 1], "the two entries are of one row"
        calls += [(N, B) if M is A else (A, N), (A, B)]
    numeric_on_a_plan((A, B), calls, "two entries")
    S = W.random_csr(700, 700, 15, 54)
    S2 = reordered(S, np.random.default_rng(55))
    T = W.CSR(S.rows, S.cols, S.rowptr, S.colidx.copy(), S.values.copy())
    numeric_on_a_plan((S, S), [(S, S), (S2, S), (S, T), (S2, S2), (T, S)], "A times A")


def test_a_row_pointer_that_leaves_room_behind_the_rows():
    """Recorded rows only, 300 places between the end of one and the start of the next: the rows themselves are the same."""
    import torch
    from paper_2404_04541_amd import binding as sg
    rng = np.random.default_rng(61)
    B = csr([np.sort(rng.choice(150, size=20, replace=False)) for _ in range(60)], 150, np.float64, 62)
    A = csr([rng.choice(60, size=10, replace=False) for _ in range(500)], 60, np.float64, 63)
    h = sg.Handle()
    dA, dB = sg.to_device(A), sg.to_device(B)
    rp, nnz, plan = sg.spgemm_symbolic(h, dA, dB)
    gap = 300
    wide = rp + gap * torch.arange(A.rows + 1, device="cuda")
    total = int(wide[-1])
    col = torch.full((total,), -1, dtype=torch.int32, device="cuda")
    val = torch.full((total,), float("nan"), dtype=torch.float64, device="cuda")
    sg.spgemm_numeric(h, plan, dA, dB, wide, col, val)
    torch.cuda.synchronize()
    assert plan.stats()["num_bin_rows"][2] == A.rows
    plan.destroy()
    keep = torch.arange(nnz, device="cuda") + gap * (torch.searchsorted(rp, torch.arange(nnz, device="cuda"), right=True) - 1)
    assert_matches_oracle(A, B, (rp.cpu().numpy(), col[keep].cpu().numpy(), val[keep].cpu().numpy()), what="gaps")


def test_numeric_phase_under_capture_on_a_kept_plan():
    """The numeric phase only enqueues kernels: a captured one follows the operands' buffers, values and order, in every replay."""
    import torch
    from paper_2404_04541_amd import binding as sg
    A, B = operands(5000, np.float64)
    rng = np.random.default_rng(71)
    stream = torch.cuda.Stream()
    h = sg.Handle(stream=stream)
    with torch.cuda.stream(stream):
        dA, dB = sg.to_device(A), sg.to_device(B)
        rp, nnz, plan = sg.spgemm_symbolic(h, dA, dB)
        col = torch.empty(nnz, dtype=torch.int32, device="cuda")
        val = torch.empty(nnz, dtype=torch.float64, device="cuda")
        sg.spgemm_numeric(h, plan, dA, dB, rp, col, val)
        stream.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=stream):
            sg.spgemm_numeric(h, plan, dA, dB, rp, col, val)
    for n, (X, Y) in enumerate([(A, B), (reordered(A, rng), B), (A, B), (A, reordered(B, rng)), (A, B)]):
        X = W.CSR(X.rows, X.cols, X.rowptr, X.colidx, X.values * (n + 1))
        for d, m in ((dA, X), (dB, Y)):
            d.colidx.copy_(torch.from_numpy(m.colidx))
            d.values.copy_(torch.from_numpy(m.values))
        col.fill_(-1)
        val.fill_(float("nan"))
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert_matches_oracle(X, Y, (rp.cpu().numpy(), col.cpu().numpy(), val.cpu().numpy()), what=f"replay {n}")
        sg.spgemm(sg.Handle(), dA, dB)   # (other work between the replays)
    plan.destroy()


@pytest.mark.parametrize("dtype", [np.float64, np.float32])
@pytest.mark.parametrize("sort_b", [True, False])
@pytest.mark.parametrize("b_rows,cols", [(400, 300), (600_000, 300), (400, 1 << 23), (600_000, 1 << 25), (400, (1 << 25) + 1), (600_000, 40_000_000)])
def test_short_rows_in_one_call(b_rows, cols, dtype, sort_b):
    """As test_short_rows; the plan of a single call has sorted words however few products there are."""
    A, B = short_operands(b_rows, cols, dtype, sort_b)
    for options in ({}, {COLUMN_LIST: 20_000}):
        assert_matches_oracle(A, B, gpu_product(A, B, via="single", options=options), what=f"rows={b_rows} cols={cols} {options}")


@pytest.mark.parametrize("entries", [10_000, (1 << 20) - 1, 1 << 20, (1 << 20) + 1])
def test_order_beside_the_rows_and_before_them(entries):
    """Up to 2^20 entries of both operands the kernel of recorded rows looks at their order beside its rows."""
    rng = np.random.default_rng(entries)
    B = csr([np.sort(rng.choice(3000, size=20, replace=False)) for _ in range(300)], 3000, np.float64, 81)
    rows = max(1, (entries - B.nnz) // 20)
    lens = np.full(rows, (entries - B.nnz) // rows)
    lens[:(entries - B.nnz) % rows] += 1
    starts = rng.integers(0, 300, size=rows)
    colidx = (np.repeat(starts, lens) + 7 * (np.arange(lens.sum()) - np.repeat(np.cumsum(lens) - lens, lens))) % 300   # (distinct in a row)
    A = W.CSR(rows, 300, np.concatenate([[0], np.cumsum(lens)]).astype(np.int64), colidx.astype(np.int32),
              W.draw_values(int(lens.sum()), -1.0, 1.0, np.float64, 82, 1))
    assert A.nnz + B.nnz == entries
    last = W.CSR(A.rows, A.cols, A.rowptr, A.colidx.copy(), A.values.copy())
    for v in (last.colidx, last.values):
        v[[-1, -2]] = v[[-2, -1]]
    numeric_on_a_plan((A, B), [(A, B), (last, B), (A, reordered(B, rng)), (A, B)], f"{entries} entries")


def rows_of_class_3(cols, dtype, short_rows):
    """Ascending B; rows of A with 600 entries of eight products each on 1000 columns spread over the matrix (193 to 1536 entries,
    more than 1536 products, tiles); short_rows: rows with a record among them, and rows of the hash class without tiles."""
    rng = np.random.default_rng(91)
    used = np.sort(rng.choice(cols, size=1000, replace=False))
    B = csr([np.sort(rng.choice(used, size=8, replace=False)) for _ in range(900)], cols, dtype, 92)
    a = [rng.choice(900, size=600, replace=False) for _ in range(60)]
    if short_rows:
        a += [rng.choice(900, size=n, replace=False) for n in (20, 24, 60, 90, 130, 190) for _ in range(20)]
    return csr(a, 900, dtype, 93), B


@pytest.mark.parametrize("dtype", [np.float64, np.float32])
@pytest.mark.parametrize("short_rows", [False, True])
@pytest.mark.parametrize("cols,options", [(1 << 19, {}), (1 << 20, {5: 0}), (3 << 18, {COLUMN_LIST: 0}), (1 << 19, {6: 100}), (24_000, {3: 256}), (2_000, {3: 256})])
def test_tiles_of_an_ascending_b_that_no_longer_ascends(cols, options, short_rows, dtype):
    """Rows of numeric class 3 by several tiles, no row of the dense classes: any order of B's entries is allowed on a kept plan.
    Options: without the block table, without the structure list, searched tiles, direct tiles."""
    A, B = rows_of_class_3(cols, dtype, short_rows)
    rng = np.random.default_rng(94)
    A2, B2 = reordered(A, rng), reordered(B, rng)
    st = numeric_on_a_plan((A, B), [(A, B), (A, B2), (A2, B), (A2, B2), (A, B)], f"{cols} columns, {options}", options=options)
    assert st["num_bin_rows"][3] >= 60 and st["num_bin_rows"][5] + st["num_bin_rows"][6] == 0 and st["dense_runs"] > 0
    assert st["dense_tiles"] >= (120 if cols > 2_000 and 6 not in options else 60)


def test_tiles_of_another_order_under_capture():
    """A captured numeric phase looks at the order in every replay."""
    import torch
    from paper_2404_04541_amd import binding as sg
    A, B = rows_of_class_3(1 << 19, np.float64, False)
    rng = np.random.default_rng(95)
    stream = torch.cuda.Stream()
    h = sg.Handle(stream=stream)
    with torch.cuda.stream(stream):
        dA, dB = sg.to_device(A), sg.to_device(B)
        rp, nnz, plan = sg.spgemm_symbolic(h, dA, dB)
        col = torch.empty(nnz, dtype=torch.int32, device="cuda")
        val = torch.empty(nnz, dtype=torch.float64, device="cuda")
        stream.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=stream):
            sg.spgemm_numeric(h, plan, dA, dB, rp, col, val)
    for n, (X, Y) in enumerate([(A, B), (A, reordered(B, rng)), (A, B), (reordered(A, rng), reordered(B, rng))]):
        for d, m in ((dA, X), (dB, Y)):
            d.colidx.copy_(torch.from_numpy(m.colidx))
            d.values.copy_(torch.from_numpy(m.values))
        col.fill_(-1)
        val.fill_(float("nan"))
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert_matches_oracle(X, Y, (rp.cpu().numpy(), col.cpu().numpy(), val.cpu().numpy()), what=f"replay {n}")
    plan.destroy()
