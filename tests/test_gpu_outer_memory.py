"""Outer products whose allocator refuses memory: what is on its way then, and that the optional memory is optional."""
import ctypes as C

import numpy as np
import pytest

import oracle
from paper_2404_04541_amd import workloads as W
from helpers import RTOL, assert_matches_oracle
from test_gpu_plan_memory import Memory

pytestmark = pytest.mark.gpu


class Outer:
    """Operands, the product from the oracle, and calls of spgemm_outer with an allocator's memory."""

    def __init__(self, A, B, capacity):
        from paper_2404_04541_amd import binding as sg
        self.sg, self.capacity, self.dtype = sg, capacity, A.values.dtype
        h = sg.Handle()
        self.a, self.b = sg.dcsc_from_csr(h, sg.to_device(A)), sg.dcsr_from_csr(h, sg.to_device(B))
        self.ref = oracle.spgemm(A, B)
        self.products = int(self.ref.ip.sum())

    def call(self, m, check=True):
        """-> the call's status, and whether the stream was idle when it returned."""
        import torch
        sa, sb, sc = self.a.struct(), self.b.struct(), self.sg.CsrStruct()
        torch.cuda.synchronize()
        rc = m.lib.spgemm_outer(m.h, C.byref(sa), C.byref(sb), self.capacity, C.byref(sc))
        idle = torch.cuda.current_stream().query()
        torch.cuda.synchronize()
        if rc == 0:
            if check:
                ref, dtype = self.ref, torch.from_numpy(np.zeros(1, self.dtype)).dtype
                get = lambda ptr, n, t: m.live[ptr][:n * t.itemsize].view(t).cpu().numpy()  # noqa: E731
                assert np.array_equal(get(sc.rowptr, sc.rows + 1, torch.int64), ref.rowptr)
                assert np.array_equal(get(sc.colidx, sc.nnz, torch.int32), ref.colidx)
                err = np.abs(get(sc.values, sc.nnz, dtype).astype(np.float64) - ref.values.astype(self.dtype).astype(np.float64))
                assert np.all(err <= RTOL[np.dtype(self.dtype)] * ref.absum)
            for ptr in (sc.rowptr, sc.colidx, sc.values):
                m.lib.spgemm_free_device(m.h, ptr)
        return rc, idle


def refuse_request(number):
    count = [0]

    def refuse(_n, _used):
        count[0] += 1
        return count[0] - 1 == number
    return refuse


@pytest.mark.parametrize("batches", [1, 2])
def test_nothing_is_on_its_way_when_a_request_is_refused(batches):
    """Every request in turn: the call goes on without it, or returns when its kernels are done (they write to memory of the host that the next
    call takes, here a product of another handle on another stream)."""
    import torch
    from paper_2404_04541_amd import binding as sg
    A = W.uniform_rows(150_000, 50_000, 8, 81, 1, np.float64)
    B = W.uniform_rows(50_000, 65_536, 5, 81, 3, np.float64)
    o = Outer(A, B, 6_000_000 // batches)
    assert o.products == 6_000_000
    X, Y = W.config3(scale=10)
    want = oracle.spgemm(X, Y)
    side = torch.cuda.Stream()
    other = sg.Handle(stream=side)
    dX, dY = sg.to_device(X), sg.to_device(Y)
    m = Memory(sg)
    assert o.call(m)[0] == 0
    m.close()
    refused = 0
    for number in range(len(m.asked)):
        m = Memory(sg, refuse_request(number))
        rc, idle = o.call(m)
        assert rc in (0, -5) and idle, number
        refused += rc != 0
        m.close()
        with torch.cuda.stream(side):
            got = sg.spgemm(other, dX, dY)
            side.synchronize()
        assert_matches_oracle(X, Y, [t.cpu().numpy() for t in (got.rowptr, got.colidx, got.values)], want)
    assert refused >= 8


def test_a_first_batch_that_is_kept_does_not_take_the_room_of_the_rest():
    """A coordinate comes hundreds of times in every batch.  Every limit at which some request just finds room or does not, down to what the call
    takes when the first batch is added up by itself."""
    from paper_2404_04541_amd import binding as sg
    A, B = W.uniform_rows(40, 2000, 1000, 65, 1, np.float32), W.uniform_rows(2000, 30, 10, 65, 3, np.float32)
    batch = 100_000
    o = Outer(A, B, batch)
    assert o.products == 4 * batch
    seen, of_that_size = [], [0]
    m = Memory(sg, lambda n, used: seen.append(used + n))
    assert o.call(m)[0] == 0
    m.close()

    def no_other_buffers(n, _used):   # (keys and values of the accumulation array, twice, then the others)
        of_that_size[0] += n == 8 * batch
        return n == 8 * batch and of_that_size[0] > 4
    m = Memory(sg, no_other_buffers)
    assert o.call(m)[0] == 0 and of_that_size[0] > 4
    least = m.most
    m.close()
    limits = {least} | {v - short for v in seen for short in (0, 1) if v - short >= least}
    assert len(limits) > 4
    for limit in sorted(limits):
        m = Memory(sg, lambda n, used: used + n > limit)
        assert o.call(m)[0] == 0, limit
        m.close()
    m = Memory(sg, lambda n, used: used + n > 32 * batch)
    assert o.call(m)[0] == -5   # (not even the accumulation array)
    m.close()


def test_a_refusal_by_the_device_leaves_no_error_behind():
    """Without an allocator of the caller's: the card has room for the accumulation array and the result, not for a second accumulation array,
    which the call then does without."""
    import torch
    from paper_2404_04541_amd import binding as sg
    A, B = W.uniform_rows(4096, 2048, 64, 83, 1, np.float32), W.uniform_rows(2048, 500, 128, 83, 3, np.float32)
    h = sg.Handle()
    a, b = sg.dcsc_from_csr(h, sg.to_device(A)), sg.dcsr_from_csr(h, sg.to_device(B))
    want = sg.spgemm(h, sg.to_device(A), sg.to_device(B))
    batch = 1 << 24
    bare = sg.Handle(torch_allocator=False)

    def call():
        sa, sb, sc = a.struct(), b.struct(), sg.CsrStruct()
        rc = bare.lib.spgemm_outer(bare.ptr, C.byref(sa), C.byref(sb), batch, C.byref(sc))
        text = bare.lib.spgemm_last_error(bare.ptr)
        nnz = int(sc.nnz)
        for ptr in (sc.rowptr, sc.colidx, sc.values):
            bare.lib.spgemm_free_device(bare.ptr, ptr)
        return rc, nnz, text
    assert call()[:2] == (0, want.nnz)   # (and what the kernels need of the device themselves is there)
    torch.cuda.empty_cache()
    room = 32 * batch + 8 * batch + (100 << 20)   # (keys of the second array find room, values do not)
    free = torch.cuda.mem_get_info()[0]
    ballast = torch.empty(free - room, dtype=torch.uint8, device="cuda")
    try:
        rc, nnz, text = call()
    finally:
        del ballast
        torch.cuda.empty_cache()
    assert (rc, nnz) == (0, want.nnz), text


@pytest.mark.parametrize("dtype", [np.float64, np.float32])
def test_a_batch_that_does_not_fit_the_limit_is_added_up_first(dtype):
    """Six batches with a coordinate some four times in each: the all array (at most 3000 components) and a batch of 12 000 reach any limit up to 15 000,
    but not the all array and the batch's different coordinates."""
    from paper_2404_04541_amd import binding as sg
    A, B = W.uniform_rows(40, 300, 180, 91, 1, dtype), W.uniform_rows(300, 75, 10, 91, 3, dtype)
    ref = oracle.spgemm(A, B)
    assert int(ref.ip.sum()) == 72_000 and ref.colidx.size == 3000
    h = sg.Handle()
    a, b = sg.dcsc_from_csr(h, sg.to_device(A)), sg.dcsr_from_csr(h, sg.to_device(B))
    for limit in (6001, 12_000, 14_999, 15_000, 15_001, 24_000, 24_001, (1 << 32) - 1):
        h.set_option(sg.OPT_MERGE_LIMIT, limit)
        c = sg.spgemm_outer(h, a, b, 12_000)
        assert np.array_equal(c.rowptr.cpu().numpy(), ref.rowptr) and np.array_equal(c.colidx.cpu().numpy(), ref.colidx), limit
        err = np.abs(c.values.cpu().numpy().astype(np.float64) - ref.values.astype(dtype).astype(np.float64))
        assert np.all(err <= RTOL[np.dtype(dtype)] * ref.absum), limit
    for limit in (2, 3000):
        h.set_option(sg.OPT_MERGE_LIMIT, limit)
        with pytest.raises(sg.SpgemmError) as e:
            sg.spgemm_outer(h, a, b, 12_000)
        assert e.value.status == -4
