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
                   'extern "C" long long counter_bytes(long long n) { return (long long)spg::sort_counter_bytes(n); }\n'
                   'extern "C" void plan(long long n, int bits, int* o) { auto p = spg::sort_plan(n, bits, false); o[0] = p.low; o[1] = p.sh.passes; o[2] = p.sh.bits; o[3] = p.sh.first_bit; o[4] = spg::sort_shape(n, bits).passes; }\n')
    lib = d / "shape.so"
    subprocess.run(["g++", "-std=c++17", "-O1", "-fPIC", "-shared", "-I", CSRC, "-o", str(lib), str(src)], check=True)
    lib = C.CDLL(str(lib))
    for f in ("ranges", "per_range", "counter_bytes"):
        getattr(lib, f).argtypes = [C.c_longlong]
    lib.plan.argtypes = [C.c_longlong, C.c_int, C.POINTER(C.c_int)]
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


def test_passes_and_buckets_sort_by_all_bits(shape):
    some = 0
    for n in (1, 2, 191, 193, 1000, 4096, 200_003, 1 << 20, 10_000_000, 12_582_912, 1 << 24, (1 << 24) + 1, 18_900_000, 1 << 27, (1 << 32) - 2):
        for bits in range(1, 63):
            o = (C.c_int * 5)()
            shape.plan(n, bits, o)
            low, passes, digit, first, plain = o
            if low == 0:
                assert first == 0 and passes == plain
                continue
            some += 1
            assert first == low and 1 <= digit <= 8 and low + passes * digit >= bits and low <= 20
            assert passes + 1 < plain                                   # (fewer steps than passes alone)
            assert 1 << (passes * digit) <= 8 * (n // 16 + 1024) and passes * digit <= 24
            if low + passes * 8 == bits: assert n >> (passes * 8) <= 512 or passes == 3
    assert some > 100
