"""Where the lanes of a recorded row read B's values in loads of four, from the kernels' own header compiled for the host: wherever a row is not
taken to be one that reaches behind the end of B, every lane's load stays inside, also of lanes that have no products to read."""
import ctypes as C
import os
import random
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2404_04541_amd", "csrc")


@pytest.fixture(scope="module")
def reads(tmp_path_factory):
    d = tmp_path_factory.mktemp("quad_reads")
    src = d / "reads.cpp"
    src.write_text('#include "quad_reads.hpp"\n'
                   'extern "C" int leaves(int lane, long long bs, int len, long long nnz) { return spg::quads_leave(lane, bs, len, nnz); }\n'
                   'extern "C" unsigned word(int src, int left, int off) { return spg::pack_quad(src, left, off); }\n'
                   'extern "C" int src_of(unsigned w) { return spg::quad_src(w); }\n'
                   'extern "C" int count_of(unsigned w) { return spg::quad_count(w); }\n'
                   'extern "C" int off_of(unsigned w) { return spg::quad_off(w); }\n')
    lib = d / "reads.so"
    subprocess.run(["g++", "-std=c++17", "-O1", "-fPIC", "-shared", "-I", CSRC, "-o", str(lib), str(src)], check=True)
    lib = C.CDLL(str(lib))
    lib.leaves.argtypes = [C.c_int, C.c_longlong, C.c_int, C.c_longlong]
    lib.word.restype = C.c_uint
    for f in ("src_of", "count_of", "off_of"):
        getattr(lib, f).argtypes = [C.c_uint]
    return lib


def wide_loads(lib, rowptr, row):
    """The first position of every lane's load of the row (B's rows `row`), or None where the row is read entry by entry."""
    nnz = rowptr[-1]
    # (lanes without an entry hold the start of the row's first)
    bs = [rowptr[row[t]] if t < len(row) else rowptr[row[0]] for t in range(64)]
    lens = [rowptr[row[t] + 1] - bs[t] if t < len(row) else 0 for t in range(64)]
    if any(lib.leaves(t, bs[t], lens[t], nnz) for t in range(64)):
        return None
    words = [lib.word(t, lens[t] - off, off) for t in range(len(row)) for off in range(0, lens[t], 4)]
    assert 0 < len(words) <= 256
    words += [0] * (-len(words) % 64)   # (idle lanes of the last round)
    out = []
    for w in words:
        out.append(bs[lib.src_of(w)] + lib.off_of(w))
        assert lib.count_of(w) <= 4
    return out


def check(lib, lens_b, row):
    rowptr = [0]
    for n in lens_b:
        rowptr.append(rowptr[-1] + n)
    at = wide_loads(lib, rowptr, row)
    if at is not None:
        assert min(at) >= 0 and max(at) + 4 <= rowptr[-1], (lens_b[-4:], row[:3])
    return at is not None


@pytest.mark.parametrize("last", [[0], [0, 0], [1, 0], [2, 0], [3, 0], [4, 0], [0, 1], [0, 3], [0, 4], [5]])
@pytest.mark.parametrize("first", [-1, -2, 0])
def test_a_first_entry_at_the_end_of_b(reads, last, first):
    lens = [5] * 999 + last
    check(reads, lens, [len(lens) + first if first else 0] + list(range(1, 41)))


def test_rows_away_from_the_end_take_wide_loads(reads):
    assert check(reads, [5] * 1000, list(range(40)))
    assert check(reads, [0] + [5] * 1000, [0] + list(range(40)))   # (an empty row far from the end)
    assert check(reads, [5] * 1000 + [0], list(range(40)) + [1000])   # (an empty row at the end that no lane reads from)


def test_rows_at_random(reads):
    rng = random.Random(7)
    wide = 0
    for _ in range(4000):
        lens = [rng.choice([0, 0, 1, 2, 3, 4, 5, 13]) for _ in range(rng.randint(1, 90))]
        row = [rng.randrange(max(0, len(lens) - 8), len(lens)) if rng.random() < 0.1 else rng.randrange(len(lens)) for _ in range(rng.randint(1, 64))]
        if sum(lens[k] for k in row):
            wide += check(reads, lens, row)
    assert wide > 100
