"""How the streaming pass is cut into shares (csrc/shares.h, compiled here for the host): every chunk once and in order, no more
shares than workgroups, and the dearest one as cheap as the best of all cuts, found by looking at them all."""
import ctypes as C
import os
import subprocess

import numpy as np
import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
SEGMENT, LEAST = 20, 16


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    so = str(tmp_path_factory.mktemp("shares") / "shares.so")
    subprocess.run(["g++", "-O2", "-std=c++17", "-shared", "-fPIC", os.path.join(HERE, "csrc", "shares_host.cpp"), "-o", so], check=True)
    return C.CDLL(so)


def _shares(lib, sizes, wgs):
    ends = np.cumsum(sizes).astype(np.uint32)
    out = np.zeros(max(int(ends[-1]) if len(ends) else 0, 1), np.uint32)
    n = lib.shares(ends.ctypes.data_as(C.c_void_p), len(ends), wgs, out.ctypes.data_as(C.c_void_p), len(out))
    assert n <= len(out)
    return out[:n].astype(int), ends.astype(int)


def _cost(first, ends):
    """Of every share: its chunks, and SEGMENT for each layer it has a part of."""
    last = np.append(first[1:], ends[-1])
    return (last - first) + SEGMENT * (np.searchsorted(ends, last - 1, side="right") - np.searchsorted(ends, first, side="right") + 1)


@pytest.mark.parametrize("sizes,wgs", [([9], 1), ([9], 256), ([16, 17], 256), ([1000], 7), ([9] * 12, 3), ([40, 9, 9, 9, 60], 4),
                                       ([100, 30, 10, 55], 5), ([33, 9, 200, 12], 2), ([64], 1)])
def test_no_cut_is_better(lib, sizes, wgs):
    first, ends = _shares(lib, sizes, wgs)
    assert first[0] == 0 and (np.diff(first) > 0).all() and first[-1] < ends[-1] and len(first) <= wgs
    n = int(ends[-1])
    layer = np.searchsorted(ends, np.arange(n), side="right")
    i, j = np.arange(n)[:, None], np.arange(1, n + 1)[None, :]
    cost = np.where(j > i, (j - i) + SEGMENT * (layer[j - 1] - layer[i] + 1), 10 ** 9)     # of the chunks i .. j - 1
    best = np.full(n + 1, 10 ** 9)
    best[0] = 0
    for _ in range(min(wgs, n)):
        best[1:] = np.minimum(best[1:], np.maximum(best[:-1, None], cost).min(axis=0))
    assert _cost(first, ends).max() <= max(int(best[n]), SEGMENT + LEAST)


@pytest.mark.parametrize("layers,wgs", [(20000, 256), (300, 256), (3, 256), (1, 1), (5000, 1)])
def test_many_layers(lib, layers, wgs):
    sizes = np.random.default_rng(layers).integers(9, 400, size=layers)
    first, ends = _shares(lib, sizes, wgs)
    assert first[0] == 0 and (np.diff(first) > 0).all() and len(first) <= wgs
    assert _cost(first, ends).max() <= max(-(-int(ends[-1] + SEGMENT * (layers + wgs)) // wgs) + SEGMENT, SEGMENT + LEAST)
    assert len(_shares(lib, [], 256)[0]) == 0
