"""Records of the allocation's candidate lists, counted on the host from the grid sizes (csrc/list_count.h): the different costs of
every row, for any cost unit."""
import ctypes as C
import os
import subprocess

import numpy as np
import pytest

HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    out = str(tmp_path_factory.mktemp("count") / "count.so")
    subprocess.run(["g++", "-O2", "-std=c++17", "-shared", "-fPIC", os.path.join(HERE, "csrc", "list_count_host.cpp"), "-o", out],
                   check=True)
    h = C.CDLL(out)
    h.count.argtypes = [C.c_void_p] + [C.c_uint64] * 5
    h.count.restype = C.c_uint64
    return h


def _plain(kt, unit, cap):
    return sum(len({-(-int(k) // unit) for k in row if -(-int(k) // unit) <= cap}) for row in kt)


def test_count_is_that_of_plain_division(lib):
    rng = np.random.default_rng(0)
    top = 0xFFF00000
    units = [1, 2, 3, 7, 8, 641, 1000, 65535, 65536, 65537, 6700417, 2**31 - 1, 2**31, 2**32 - 5, 2**32 - 1, 2**32, 2**32 + 1, 2**40 + 3, 2**61]
    for _ in range(400):
        L, J = int(rng.integers(1, 6)), int(rng.integers(1, 65))
        unit = int(rng.choice(units)) if rng.random() < 0.6 else int(10 ** rng.uniform(0, 10))
        kt = np.sort(np.minimum(top, np.maximum(1, 10 ** rng.uniform(0, 9.7, size=(L, J)))).astype(np.uint32), axis=1)
        near = np.clip(rng.integers(0, 50, size=(L, J)) * unit + rng.integers(-1, 2, size=(L, J)), 1, top)      # around multiples
        if unit < 2**40 and rng.random() < 0.5:
            kt = np.sort(near.astype(np.uint32), axis=1)
        kt = np.ascontiguousarray(kt)
        cap = int(rng.choice([1, 5, 4096, 2**33]))
        want = _plain(kt, unit, cap)
        assert lib.count(kt.ctypes.data, L, J, unit, cap, 1 << 40) == want, (unit, cap)
        if want > 3:                               # stops once the limit is passed
            got = lib.count(kt.ctypes.data, L, J, unit, cap, 3)
            assert 3 < got <= want
