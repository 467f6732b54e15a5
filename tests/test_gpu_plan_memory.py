"""Products whose allocator refuses some of the plan's optional memory: which parts go, and that the rest still gives C."""
import ctypes as C

import numpy as np
import pytest

import oracle
from paper_2404_04541_amd import workloads as W
from helpers import assert_matches_oracle

pytestmark = pytest.mark.gpu


class Memory:
    """An allocator that logs what it is asked for and refuses what `refuse(bytes, bytes in use)` says."""

    def __init__(self, sg, refuse=lambda n, used: False):
        import torch
        self.sg, self.live, self.asked, self.used, self.most = sg, {}, [], 0, 0

        def alloc(_ctx, n):
            self.asked.append(n)
            if refuse(n, self.used):
                return None
            t = torch.empty(max(int(n), 1), dtype=torch.uint8, device="cuda")
            self.live[t.data_ptr()] = t
            self.used += n
            self.most = max(self.most, self.used)
            return t.data_ptr()

        def free(_ctx, ptr):
            self.used -= self.live.pop(ptr).numel()

        self.cb = (sg.ALLOC_FN(alloc), sg.FREE_FN(free))
        self.struct = sg.AllocatorStruct(self.cb[0], self.cb[1], None)
        self.lib = sg.load_library()
        self.h = C.c_void_p()
        assert self.lib.spgemm_create(C.byref(self.h), None, C.byref(self.struct)) == 0

    def close(self):
        assert not self.live and self.lib.spgemm_destroy(self.h) == 0

    def product(self, A, B, column_list=1, blocks=0):
        """spgemm, or spgemm_pipelined in so many blocks; compared with the oracle.  -> the call's status."""
        import torch
        sg, lib = self.sg, self.lib
        assert lib.spgemm_set_option(self.h, sg.OPT_COLUMN_LIST, column_list) == 0
        dA, dB = sg.to_device(A), sg.to_device(B)
        sa, sb = dA.struct(), dB.struct()
        parts = (sg.CsrStruct * max(blocks, 1))()
        first = (C.c_int64 * (blocks + 1))()
        if blocks:
            rc = lib.spgemm_pipelined(self.h, C.byref(sa), C.byref(sb), blocks, parts, first)
        else:
            rc = lib.spgemm(self.h, C.byref(sa), C.byref(sb), C.byref(parts[0]))
        torch.cuda.synchronize()
        if rc != 0:
            return rc
        rp, col, val = [np.zeros(1, np.int64)], [], []
        for c in parts:
            get = lambda ptr, n, t: self.live[ptr][:n * t.itemsize].view(t) if n else torch.empty(0, dtype=t, device="cuda")  # noqa: E731
            rp.append(get(c.rowptr, c.rows + 1, torch.int64).cpu().numpy()[1:] + rp[-1][-1])
            col.append(get(c.colidx, c.nnz, torch.int32).cpu().numpy())
            val.append(get(c.values, c.nnz, dA.values.dtype).cpu().numpy())
            for ptr in (c.rowptr, c.colidx, c.values):
                if ptr:
                    lib.spgemm_free_device(self.h, ptr)
        assert_matches_oracle(A, B, (np.concatenate(rp), np.concatenate(col), np.concatenate(val)))
        return 0

    def phases(self, A, B):
        """Both phases by themselves -> stats, and what was asked for by the symbolic one."""
        import torch
        sg, lib = self.sg, self.lib
        dA, dB = sg.to_device(A), sg.to_device(B)
        sa, sb = dA.struct(), dB.struct()
        rp = torch.empty(A.rows + 1, dtype=torch.int64, device="cuda")
        nnz, plan, st = C.c_int64(), C.c_void_p(), sg.StatsStruct()
        assert lib.spgemm_symbolic(self.h, C.byref(sa), C.byref(sb), rp.data_ptr(), C.byref(nnz), C.byref(plan)) == 0, lib.spgemm_last_error(self.h)
        col = torch.empty(nnz.value, dtype=torch.int32, device="cuda")
        val = torch.empty(nnz.value, dtype=dA.values.dtype, device="cuda")
        assert lib.spgemm_numeric(self.h, plan, C.byref(sa), C.byref(sb), rp.data_ptr(), col.data_ptr(), val.data_ptr()) == 0
        torch.cuda.synchronize()
        assert lib.spgemm_get_stats(plan, C.byref(st)) == 0
        assert lib.spgemm_plan_destroy(plan) == 0
        assert_matches_oracle(A, B, (rp.cpu().numpy(), col.cpu().numpy(), val.cpu().numpy()))
        return st


def test_the_structure_list_is_kept_when_the_rest_is_refused():
    from paper_2404_04541_amd import binding as sg
    A, B = W.config3(scale=13)
    m = Memory(sg)
    st = m.phases(A, B)
    m.close()
    whole = m.asked[-1]   # (the optional part is the last thing a plan asks for)
    assert st.plan_list_bytes > 0 and whole > st.plan_list_bytes
    m = Memory(sg, lambda n, used: n == whole)
    less = m.phases(A, B)
    m.close()
    assert less.plan_list_bytes == st.plan_list_bytes and less.plan_list_used > 0
    assert less.plan_bytes == st.plan_bytes - (whole - st.plan_list_bytes)


def described(rows=200_000):
    """B's row pointer is larger than an L2 slice and rows are short: the row count describes the entries of A (8 bytes each)."""
    A = W.uniform_rows(rows, 600_000, 8, 71, 1)
    return A, W.uniform_rows(600_000, 5000, 4, 72, 3)


def test_descriptions_are_part_of_the_optional_memory():
    from paper_2404_04541_amd import binding as sg
    A, B = described()
    desc = A.nnz * 8
    for column_list, want in ((1, True), (0, False), (4096, False), (desc - 1, False), (desc, True)):
        m = Memory(sg)
        assert m.product(A, B, column_list) == 0
        assert (desc in m.asked) == want, column_list
        m.close()
    m = Memory(sg)
    assert m.product(A, B, blocks=3) == 0
    assert max(m.asked) < desc or desc not in m.asked   # (a block's positions are those of the whole matrix)
    m.close()
    m = Memory(sg, lambda n, used: n == desc)
    assert m.product(A, B) == 0
    m.close()


def test_c_is_asked_for_again_without_any_optional_memory():
    from paper_2404_04541_amd import binding as sg
    A, B = described()
    m = Memory(sg)
    assert m.product(A, B, 0) == 0
    least = m.most   # what the product cannot do without
    m.close()
    m = Memory(sg)
    assert m.product(A, B) == 0 and m.most > least
    m.close()
    m = Memory(sg, lambda n, used: used + n > least)
    assert m.product(A, B) == 0 and A.nnz * 8 in m.asked
    m.close()


def test_the_plan_gives_the_descriptions_back_when_its_lists_find_no_room():
    from paper_2404_04541_amd import binding as sg
    A, B = described(20_000)
    long_rows = W.uniform_rows(50, 600_000, 2000, 73, 1)   # (dense: 8000 products)
    A = W.CSR(A.rows + 50, A.cols, np.concatenate([A.rowptr, A.rowptr[-1] + long_rows.rowptr[1:]]),
              np.concatenate([A.colidx, long_rows.colidx]), np.concatenate([A.values, long_rows.values]))
    m = Memory(sg)
    m.phases(A, B)
    asked = m.asked
    m.close()
    desc = A.nnz * 8
    lists = asked[asked.index(desc) + 1]   # tile and run lists, the block table: the plan cannot do without
    before = sum(asked[:asked.index(desc)])
    m = Memory(sg, lambda n, used: used + n > before + max(desc, lists))
    m.phases(A, B)
    assert lists in m.asked and m.asked.count(lists) == 2
    m.close()


@pytest.mark.parametrize("case", ["graph", "short rows"])
def test_row_blocks_go_on_without_the_optional_memory(case):
    from paper_2404_04541_amd import binding as sg
    A, B = W.config3(scale=13) if case == "graph" else (W.uniform_rows(30_000, 4000, 20, 74, 1), W.uniform_rows(4000, 3000, 20, 75, 3))
    m = Memory(sg)
    assert m.product(A, B, 0, blocks=4) == 0
    least = m.most
    m.close()
    m = Memory(sg)
    assert m.product(A, B, blocks=4) == 0 and m.most > least
    m.close()
    m = Memory(sg, lambda n, used: used + n > least)
    assert m.product(A, B, blocks=4) == 0
    m.close()
    m = Memory(sg, lambda n, used: used + n > least // 2)
    assert m.product(A, B, blocks=4) == -5   # (too little even so: an error, and nothing is left behind)
    m.close()


@pytest.mark.parametrize("alike", [False, True])
def test_records_find_room_in_a_limit(alike):
    """A limit that holds four bytes for every row of A and the records of the rows that can have one (1792 bytes each), but not eight bytes a
    row.  Rows that are not alike have no use for more; rows that are do without being taken for it."""
    from paper_2404_04541_amd import binding as sg
    rng = np.random.default_rng(5)
    rows, recorded = 100_000, 40
    d = np.zeros(rows, np.int64)
    d[:recorded] = 30
    rp = np.concatenate([[0], np.cumsum(d)])
    cols = np.concatenate([np.arange(30) + i if alike else np.sort(rng.choice(500, 30, replace=False)) for i in range(recorded)])
    A = W.CSR(rows, 500, rp, cols.astype(np.int32), rng.standard_normal(cols.size))
    B = W.CSR(500, 700, np.arange(501, dtype=np.int64) * 8, ((np.arange(500)[:, None] + np.arange(8)) % 700).ravel().astype(np.int32), rng.standard_normal(4000))
    map_bytes, record_bytes = -(-rows * 4 // 256) * 256, recorded * 1792
    for limit, maps in ((map_bytes - 1, 0), (map_bytes + record_bytes, 1), (2 * map_bytes + record_bytes, 1 + alike), (1, 1 + alike)):
        m = Memory(sg)
        m.lib.spgemm_set_option(m.h, sg.OPT_COLUMN_LIST, limit)
        m.phases(A, B)
        m.close()
        assert m.asked[1:] == ([maps * map_bytes + record_bytes] if maps else []), limit   # (behind what the plan cannot do without)
