"""Arithmetic of a workgroup's share of a layer in the streaming pass (csrc/segment.h, compiled here for the host).  How far it
goes with one histogram: no entry may ever count past 2^20 - 1, whatever the chunks hold and whichever wave comes first.  How
the space for its candidates is handed out: inside the share's slice, and enough for the eighth of a layer that may spill."""
import ctypes as C
import os
import subprocess

import numpy as np
import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
MAX_COUNT, CHUNK, OPEN = 0xFFFFF, 1024, 32


@pytest.fixture(scope="module")
def seg(tmp_path_factory):
    lib = str(tmp_path_factory.mktemp("segment") / "segment.so")
    subprocess.run(["g++", "-O2", "-std=c++17", "-shared", "-fPIC", "-pthread", os.path.join(HERE, "csrc", "segment_host.cpp"),
                    "-o", lib], check=True)
    return C.CDLL(lib)


def _limit_after(seg, seg_end, allowed, taken, most):
    out = (C.c_uint32 * 2)()
    seg.limit_after(seg_end, allowed, taken, most, OPEN, out)
    return out[0], bool(out[1])


@pytest.mark.parametrize("over", [1, 7, 16, 17, 32, 200])
@pytest.mark.parametrize("ahead", [0, 1, 16, 32])
def test_the_last_chunks_of_a_segment_need_room_like_any_others(seg, over, ahead):
    """A segment that ends soon after the limit of its first 1023 chunks, all of one value; the other waves have taken chunks up
    to its end and beyond while this one reads, and up to thirty-two of them are still to be counted."""
    allowed = 1023
    seg_end = allowed + over
    for counted in range(allowed - 33, allowed + 1):
        taken = max(seg_end, allowed) + ahead
        end, on = _limit_after(seg, seg_end, allowed, taken, counted * CHUNK)
        if on:
            assert (counted + OPEN) * CHUNK <= MAX_COUNT and end == seg_end, (counted, taken)


def test_an_extension_never_lets_an_entry_overflow(seg):
    rng = np.random.default_rng(1)
    for _ in range(20000):
        allowed = int(rng.integers(1023, 6000))
        seg_end = allowed + int(rng.choice([1, 5, 16, 33, 64, 128, 1000, 5000]))
        taken = allowed + int(rng.integers(-64, 48))
        most = int(rng.choice([0, MAX_COUNT, MAX_COUNT - 31 * CHUNK, MAX_COUNT - 32 * CHUNK, MAX_COUNT - 33 * CHUNK,
                               int(rng.integers(0, MAX_COUNT + 1))]))
        end, on = _limit_after(seg, seg_end, allowed, taken, most)
        if on:
            assert most + (OPEN + max(0, end - taken)) * CHUNK <= MAX_COUNT, (allowed, seg_end, taken, most)
            assert end == seg_end or end >= allowed + 128


@pytest.mark.parametrize("chunks", [1024, 1030, 1039, 1200, 4954])
@pytest.mark.parametrize("fullest", [1024, 512, 64, 8])
def test_sixteen_waves_walk_a_segment(seg, chunks, fullest):
    """Threads in the place of waves, with the limit's code as the kernel has it.  Every chunk is counted once, no entry overflows,
    all waves end a stretch at the same chunk, and a stretch goes on for as long as its fullest entry has room."""
    rest = 1024 - fullest
    per = [fullest] + [rest // 16] * 16
    out = (C.c_uint32 * 4)()
    for spin in (0, 20, 200):
        seg.walk(16, chunks, (C.c_uint32 * len(per))(*per), len(per), spin, out)
        stretches, most, counted, apart = out[:]
        assert counted == chunks and apart == 0 and most <= MAX_COUNT, (spin, out[:])
        # a limit seen to 64 chunks ahead stays where the room, less the 32 chunks under way, does not reach 128 beyond it
        least = min((MAX_COUNT - (64 + OPEN + 128 + 2) * CHUNK) // max(per), chunks)
        assert stretches <= -(-chunks // max(least, 1023)), (spin, out[:], least)


def _spill(seg, region, first_chunk, counts, order):
    n = len(counts)
    out = (C.c_uint32 * 3)()
    seg.spill(C.c_uint64(region), first_chunk, n, (C.c_uint32 * n)(*[int(x) for x in counts]), (C.c_uint32 * n)(*[int(x) for x in order]), out)
    assert first_chunk * 168 <= out[0] and out[1] <= (first_chunk + n) * 168, (region, first_chunk, out[:])
    return bool(out[2])


def test_short_slices_hold_any_chunks_of_up_to_168_candidates(seg):
    rng = np.random.default_rng(2)
    for chunks in range(1, 17):                    # a wave each
        for region in (0, 8, 2048 + 168 * 9):
            for first in range(0, 5):
                for counts in ([168] * chunks, [129] * chunks, [64] * chunks, [1] * chunks, rng.integers(0, 169, size=chunks),
                               rng.integers(120, 169, size=chunks)):
                    assert _spill(seg, region, first, counts, range(chunks)), (chunks, region, first, counts)


@pytest.mark.parametrize("chunks", [1, 2, 3, 5, 9, 16, 17, 40, 127, 128, 129, 255, 256, 257, 511, 512, 513, 2000])
def test_a_slice_holds_an_eighth_of_its_entries(seg, chunks):
    """Counts as an eighth of independent entries gives them, and uneven ones of the same mean."""
    rng = np.random.default_rng(chunks)
    for trial in range(300 if chunks < 600 else 30):
        region, first = int(rng.integers(0, 1 << 20)) * 8, int(rng.integers(0, 1000))
        even = rng.binomial(1024, 0.125, size=chunks)
        assert even.max() > 168 or _spill(seg, region, first, even, np.arange(chunks) % 16), (chunks, region, first)
        if chunks >= 40:
            uneven = np.where(rng.random(chunks) < 0.4, rng.integers(0, 65, size=chunks), rng.integers(100, 260, size=chunks))
            if uneven.sum() <= 112 * chunks:
                assert _spill(seg, region, first, uneven, rng.integers(0, 16, size=chunks)), (chunks, region, first, uneven.sum())
