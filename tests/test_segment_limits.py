"""How far a workgroup of the streaming pass goes with one histogram (csrc/segment.h, compiled here for the host): no entry may
ever count past 2^20 - 1, whatever the chunks hold and whichever wave comes first."""
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
