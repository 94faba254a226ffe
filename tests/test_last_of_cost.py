"""A segment's first layer stores its entries side by side, a lane each: whatever the lanes' order, a cell ends up with the least
error of its cost, and has been stored once (csrc/last_of_cost.h, compiled here for the host, on lists as the allocation keeps
them of tables whose errors fall and of ones whose errors do not)."""
import ctypes as C
import os
import subprocess

import numpy as np
import pytest

HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    so = str(tmp_path_factory.mktemp("row") / "row.so")
    subprocess.run(["g++", "-O2", "-std=c++17", "-shared", "-fPIC", os.path.join(HERE, "csrc", "last_of_cost_host.cpp"), "-o", so], check=True)
    return C.CDLL(so)


def _kept(w, e):
    """The entries of a list: the last member of every run of equal costs and non-increasing errors, where it is less than all before."""
    starts = [j for j in range(len(w)) if j == 0 or w[j] != w[j - 1] or not e[j] <= e[j - 1]]
    ends = [s - 1 for s in starts[1:]] + [len(w) - 1]
    out, least = [], np.inf
    for s, t in zip(starts, ends):
        if s == 0 or e[t] < least:
            out.append((w[s], e[t]))
        least = min(least, e[t])
    return out


@pytest.mark.parametrize("falling", [True, False])
def test_any_order_of_lanes_gives_the_least_error(lib, falling):
    rng = np.random.default_rng(int(falling))
    same_cost = 0
    for _ in range(300):
        J = int(rng.integers(1, 65))
        w = np.sort(rng.integers(0, max(1, J // 3), size=J))
        w -= w[0]
        e = rng.integers(0, 8, size=J).astype(np.float64) + rng.random(J) * (rng.random() < 0.5)
        if falling:
            e = np.sort(e)[::-1]
        kept = _kept(w, e)
        n = len(kept)
        same_cost += n - len({c for c, _ in kept})
        costs, errors = np.array([c for c, _ in kept], np.uint32), np.array([x for _, x in kept])
        want = np.full(int(w[-1]) + 1, np.inf)
        for c, x in kept:
            want[c] = min(want[c], x)
        for order in (np.arange(n), np.arange(n)[::-1], rng.permutation(n)):
            row, order = np.full(int(w[-1]) + 1, np.inf), np.ascontiguousarray(order, dtype=np.uint32)
            stores = lib.store_row(costs.ctypes.data_as(C.c_void_p), errors.ctypes.data_as(C.c_void_p), n, order.ctypes.data_as(C.c_void_p),
                                   row.ctypes.data_as(C.c_void_p))
            assert np.array_equal(row, want) and stores == len(set(costs.tolist()))
    assert (same_cost == 0) == falling              # the case that it is about is there
