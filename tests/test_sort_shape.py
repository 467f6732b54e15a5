"""How the radix sort is cut, from the library's own header compiled for the host: the counters sized for n entries hold the
counters of every shorter sort (an outer product's last batch is sorted in the room made for a full one)."""
import ctypes as C
import os
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2404_04541_amd", "csrc")
TILE, BINS = 8192, 256


@pytest.fixture(scope="module")
def shape(tmp_path_factory):
    d = tmp_path_factory.mktemp("sort_shape")
    src = d / "shape.cpp"
    src.write_text('#include "sort_shape.hpp"\n'
                   'extern "C" int ranges(long long n) { return spg::sort_shape(n, 8).ranges; }\n'
                   'extern "C" long long per_range(long long n) { return spg::sort_shape(n, 8).per_range; }\n'
                   'extern "C" long long counter_bytes(long long n) { return (long long)spg::sort_counter_bytes(n); }\n')
    lib = d / "shape.so"
    subprocess.run(["g++", "-std=c++17", "-O1", "-fPIC", "-shared", "-I", CSRC, "-o", str(lib), str(src)], check=True)
    lib = C.CDLL(str(lib))
    for f in ("ranges", "per_range", "counter_bytes"):
        getattr(lib, f).argtypes = [C.c_longlong]
    lib.per_range.restype = lib.counter_bytes.restype = C.c_longlong
    return lib


def test_counters_hold_those_of_every_shorter_sort(shape):
    most = 0
    for tiles in range(1, 5000):
        for n in (tiles * TILE - TILE + 1, tiles * TILE):
            assert 1 <= shape.ranges(n) <= 1024 and shape.ranges(n) * shape.per_range(n) >= n
            most = max(most, (shape.ranges(n) + 1) * BINS * 4)   # counters of the digits' totals, then one per range and digit
            assert shape.counter_bytes(n) >= most, f"{n} entries"


@pytest.mark.parametrize("full,last", [(10_000_000, 8_000_000), (8_400_000, 8_300_000), (20_000_000, 16_700_000), (1 << 24, (1 << 24) - 1)])
def test_room_of_a_full_batch_holds_a_shorter_one(shape, full, last):
    assert shape.counter_bytes(full) >= (shape.ranges(last) + 1) * BINS * 4
