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
