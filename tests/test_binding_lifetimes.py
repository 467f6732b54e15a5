"""Handles and plans of the binding end in an order that the library allows, whoever ends them (no GPU: the library's own calls
are recorded, not made)."""
import ctypes as C
import gc
import os
import weakref

import pytest


@pytest.fixture
def sg():
    from paper_2404_04541_amd import binding
    if not os.path.exists(binding.LIB_PATH):
        from paper_2404_04541_amd.build import build_library
        build_library()
    gc.disable()
    yield binding
    gc.enable()


class Recorder:
    """In the library's place: remembers which of its calls ended what."""

    def __init__(self, lib):
        self.lib, self.calls = lib, []

    def spgemm_plan_destroy(self, ptr):
        self.calls.append(("plan", ptr.value))

    def spgemm_destroy(self, ptr):
        self.calls.append(("handle",))
        return self.lib.spgemm_destroy(ptr)

    def spgemm_get_stats(self, ptr, out):
        return -1 if ptr is None else 0

    def spgemm_last_error(self, ptr):
        return b""


def handle_with_plans(sg, n):
    h = sg.Handle()
    h.lib = Recorder(h.lib)
    return h, h.lib.calls, [sg.Plan(h, C.c_void_p(0x1000 + i), 5) for i in range(n)]


@pytest.mark.parametrize("torch_allocator", [True, False])
def test_a_handle_that_nobody_refers_to_is_gone_without_the_collector(sg, torch_allocator):
    h = sg.Handle(torch_allocator=torch_allocator)
    gone = weakref.ref(h)
    del h
    assert gone() is None


def test_a_plan_keeps_its_handle(sg):
    h, calls, (p,) = handle_with_plans(sg, 1)
    del h
    assert calls == []
    del p
    assert calls == [("plan", 0x1000), ("handle",)]


def test_a_plan_is_destroyed_once(sg):
    h, calls, (p, q) = handle_with_plans(sg, 2)
    p.destroy()
    p.destroy()
    assert calls == [("plan", 0x1000)] and p.ptr is None and q.ptr.value == 0x1001
    del p, q, h
    assert calls == [("plan", 0x1000), ("plan", 0x1001), ("handle",)]


def test_closing_a_handle_destroys_its_plans_first(sg):
    h, calls, plans = handle_with_plans(sg, 2)
    h.close()
    assert sorted(calls[:2]) == [("plan", 0x1000), ("plan", 0x1001)] and calls[2:] == [("handle",)]
    with pytest.raises(sg.SpgemmError):
        plans[0].stats()
    for p in plans:
        p.destroy()
    h.close()
    assert len(calls) == 3


@pytest.mark.parametrize("handle_first", [True, False])
def test_a_handle_and_its_plans_collected_together(sg, handle_first):
    """As in the frame of a failed call that a traceback keeps: the collector finalises in the order of creation, handle first."""
    h, calls, plans = handle_with_plans(sg, 3)
    cycle = [h, plans] if handle_first else [plans, h]
    cycle.append(cycle)
    h.cycle = cycle
    del h, plans, cycle
    gc.collect()
    assert sorted(calls[:3]) == [("plan", 0x1000 + i) for i in range(3)] and calls[3:] == [("handle",)]
