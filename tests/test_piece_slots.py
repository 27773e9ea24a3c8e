"""The slots of a split batch and the pieces that begin in them (csrc/piece_slots.h), compiled for the CPU with a wave of 64
lanes and compared with the rules said plainly: string s has the slots from s + offsets[s] // 896 on, one for each 896
bytes begun and one at least; a piece begins at its string's first byte and at the last cut within the 128 bytes up to
every 896th, a slot without one is void, and the piece before it runs on.  Both ways of finding them: listed, and a wave a slot."""
import ctypes
import os
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
TARGET, WINDOW, MAX_STRING = 896, 128, 65536
COVER_REST, COVER_FIRST = 0x40, 0x80
UNSET = -(1 << 20)


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    out = str(tmp_path_factory.mktemp("slots") / "slots.so")
    subprocess.check_call(["g++", "-O1", "-std=c++20", "-shared", "-fPIC", "-o", out,
                           "-I", os.path.join(ROOT, "paper_2507_11941_amd", "csrc"),
                           os.path.join(ROOT, "tests", "piece_slots_driver.cpp")])
    return ctypes.CDLL(out)


def ptr(a):
    return ctypes.c_void_p(a.ctypes.data if a is not None else None)


def slots(lib, data, offsets, cover, cut, steps_each):
    """cut: bool [256, 256]; returns (string, begin, length) of every slot."""
    bits = np.packbits(cut.T.reshape(-1), bitorder="little").view(np.uint32).copy()       # bit a + 256 b
    n = len(offsets) - 1 + int(offsets[-1]) // TARGET
    string, begin, length = np.full(n, UNSET, np.int32), np.full(n, UNSET, np.int64), np.full(n, UNSET, np.int32)
    lib.piece_slots(ptr(data), ptr(offsets), len(offsets) - 1, ptr(cover), ptr(bits), TARGET, MAX_STRING,
                    ctypes.c_uint32(n), ctypes.c_uint32(steps_each), ptr(string), ptr(begin), ptr(length))
    return string, begin, length


def expected(data, offsets, cover, cut):
    n = len(offsets) - 1 + int(offsets[-1]) // TARGET
    string, begin, length = np.full(n, -1, np.int32), np.full(n, -1, np.int64), np.zeros(n, np.int32)

    def is_cut(q):
        if cover is None:
            return cut[data[q - 1], data[q]]
        return (cut[data[q - 1], data[q]] or cover[q - 1] or cover[q]) and cover[q] != COVER_REST

    for s, (a, b) in enumerate(zip(offsets[:-1].tolist(), offsets[1:].tolist())):
        base = s + a // TARGET
        string[base] = s
        if b - a > MAX_STRING:
            continue
        pieces = [(base, a)]
        for i in range(1, -(-(b - a) // TARGET)):
            t = a + i * TARGET
            at = next((q for q in range(t, t - WINDOW, -1) if is_cut(q)), None)
            if at is not None:
                pieces.append((base + i, at))
        end_slot = base + max(-(-(b - a) // TARGET), 1)
        for (g, at), (until, end) in zip(pieces, pieces[1:] + [(end_slot, b)]):
            begin[g], length[g] = at, end - at
            for h in range(g + 1, until):
                length[h] = g - h
    return string, begin, length


def text(rng, n, runs):
    """Words of `a` to `z` with a cut before each space; `runs`: some long stretches of one letter, without a cut."""
    data = rng.integers(97, 123, size=n).astype(np.uint8)
    ends = np.cumsum(rng.integers(2, 13, size=n // 2 + 1))
    data[ends[ends < n]] = 32
    for _ in range(runs if n > 100 else 0):
        at = int(rng.integers(0, n - 50))
        data[at:at + int(rng.integers(50, 6 * TARGET))] = 101
    return data


CUT = np.zeros((256, 256), bool)
CUT[97:123, 32] = True

BATCHES = {
    "one": [5000], "one long": [65536], "empty": [0], "empties": [0] * 70, "short": [3] * 200,
    "edges": [895, 896, 897, 1792, 1793, 0, 1, 2687, 2688, 2689], "too long": [300, 65537, 5, 70000, 900],
    "63 slots": [63 * 896], "64 slots": [64 * 896], "65 slots": [65 * 896, 10], "mixed": [0, 0, 4000, 20, 0, 17000, 1, 1, 896] * 5,
}


@pytest.mark.parametrize("steps_each", [0, 1, 3])
@pytest.mark.parametrize("specials", [False, True])
@pytest.mark.parametrize("runs", [0, 8])
@pytest.mark.parametrize("lens", BATCHES.values(), ids=BATCHES.keys())
def test_slots(lib, lens, runs, specials, steps_each):
    rng = np.random.default_rng(len(lens) + sum(lens) + runs)
    offsets = np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)
    data, cover = text(rng, int(offsets[-1]), runs), None
    if specials:
        cover = np.zeros(len(data) + 16, np.uint8)
        for at in range(500, len(data) - 10, 430):               # marks of five bytes, some on the nominal starts
            at += int(rng.integers(0, 60))
            if at + 5 <= len(data):
                cover[at], cover[at + 1:at + 5] = COVER_FIRST, COVER_REST
    got = slots(lib, data, offsets, cover, CUT, steps_each)
    for what, g, e in zip(("string", "begin", "length"), got, expected(data, offsets, cover, CUT)):
        assert np.array_equal(g, e), (what, np.flatnonzero(g != e)[:5], g[g != e][:5], e[g != e][:5])


@pytest.mark.parametrize("steps_each", [0, 1, 3])
@pytest.mark.parametrize("skipped", [100, 2000, 130 * TARGET + 17])
def test_offsets_that_begin_later(lib, skipped, steps_each):
    """A window of a longer offsets array: the slots below the first string's are void, and nothing is read for them."""
    rng = np.random.default_rng(skipped)
    offsets = skipped + np.concatenate([[0], np.cumsum([700, 5000, 0, 66000, 30, 2000])]).astype(np.int64)
    data = text(rng, int(offsets[-1]), 4)
    got = slots(lib, data, offsets, None, CUT, steps_each)
    for what, g, e in zip(("string", "begin", "length"), got, expected(data, offsets, None, CUT)):
        assert np.array_equal(g, e), (what, np.flatnonzero(g != e)[:5], g[g != e][:5], e[g != e][:5])


def test_small_batches_leave_no_item_out(lib):
    """Batches without a list: every slot has a wave, and no workgroup of the kernel that does the rest, which takes every
    grid-th of what is left, gets more than the sixteen it has room for -- however few fit the device."""
    lib.small_batch.argtypes = [ctypes.c_int64] * 3
    lib.small_batch.restype = ctypes.c_bool
    for resident in (512, 4096, 8192):
        for rest_grid in (1, 31, 32, 255, 256, 768):
            fits = [slots for slots in range(1, 5000) if lib.small_batch(slots, resident, rest_grid)]
            assert fits == list(range(1, min(resident, 16 * rest_grid, 4096) + 1))
            assert max(-(-slots // min(rest_grid, slots)) for slots in fits) <= 16
