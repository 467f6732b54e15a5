"""What a plan takes of the free memory, from the library's own header compiled for the host: a C that fits beside the structure
list fits beside the order of the short rows as well."""
import ctypes as C
import os
import random
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2404_04541_amd", "csrc")
GB = float(1 << 30)


@pytest.fixture(scope="module")
def room(tmp_path_factory):
    d = tmp_path_factory.mktemp("plan_room")
    src = d / "room.cpp"
    src.write_text('#include "plan_room.hpp"\n'
                   'extern "C" void room(const double* in, double* out) {\n'
                   '  const spg::PlanRoom r = spg::plan_room(in[0], in[1], in[2], in[3], in[4], in[5]);\n'
                   '  out[0] = r.list; out[1] = r.shorts; out[2] = r.desc;\n}\n')
    lib = d / "room.so"
    subprocess.run(["g++", "-std=c++17", "-O1", "-fPIC", "-shared", "-I", CSRC, "-o", str(lib), str(src)], check=True)
    lib = C.CDLL(str(lib))

    def call(*args):
        out = (C.c_double * 3)()
        lib.room((C.c_double * 6)(*args), out)
        return tuple(out)
    return call


def test_c_fits_where_it_fitted_beside_the_list_alone(room):
    rng = random.Random(3)
    byte = lambda lo, hi: float(int(2.0 ** rng.uniform(lo, hi)))  # noqa: E731  (whole bytes: their sums are exact)
    size = lambda: rng.choice([0.0, byte(10, 39)])  # noqa: E731
    for _ in range(20000):
        free, list_want, short_want, c_most = byte(24, 39), size(), size(), size()
        asked = rng.choice([1e30, byte(12, 38)])
        desc = rng.choice([0.0, float(int(free * rng.random()))])   # (of the free memory, the descriptions have been taken)
        took, shorts, kept = room(free - desc, list_want, short_want, desc, c_most, asked)
        alone = min(list_want, free / 3, asked)
        shorts += desc if kept else 0.0
        assert 0 <= shorts <= min(short_want + desc, free / 4, asked) * (1 + 1e-12) and 0 <= took <= alone
        for c in (c_most, c_most * rng.random()):
            if c <= free - alone:
                assert c <= (free - took - shorts) * (1 + 1e-12)


@pytest.mark.parametrize("free,list_want,short_want,desc,c_most,want", [
    (200 * GB, 0, 4 * GB, 0, 18 * GB, (0, 4 * GB, 0)),                 # a stencil with room for everything
    (20 * GB, 0, 4 * GB, 0, 18 * GB, (0, 2 * GB, 0)),                  # C first
    (20 * GB, 0, 4 * GB, 0, 25 * GB, (0, 0, 0)),
    (280 * GB, 84 * GB, 2 * GB, 0, 168 * GB, (84 * GB, 2 * GB, 0)),
    (200 * GB, 84 * GB, 2 * GB, 0, 168 * GB, (200 * GB / 3 - 2 * GB, 2 * GB, 0)),   # a graph's short rows: out of the list
    (200 * GB, 0, 4 * GB, 3 * GB, 18 * GB, (0, 4 * GB, 1)),
    (17 * GB, 0, 4 * GB, 3 * GB, 18 * GB, (0, 2 * GB, 0)),             # the descriptions make room
    (20 * GB, 0, 40 * GB, 8 * GB, 1 * GB, (0, 7 * GB, 0)),             # more than a quarter
    (20 * GB, 0, 40 * GB, 4 * GB, 1 * GB, (0, 2 * GB, 1)),             # a quarter together
])
def test_shares(room, free, list_want, short_want, desc, c_most, want):
    assert room(free, list_want, short_want, desc, c_most, 1e30) == pytest.approx(want)


def test_the_callers_limit_holds_for_the_short_rows_together(room):
    assert room(200 * GB, 84 * GB, 4 * GB, 1 * GB, 18 * GB, 2 * GB) == pytest.approx((2 * GB, 1 * GB, 1))
    assert room(200 * GB, 84 * GB, 4 * GB, 3 * GB, 18 * GB, 2 * GB) == pytest.approx((2 * GB, 2 * GB, 0))
