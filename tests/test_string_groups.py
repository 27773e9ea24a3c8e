"""The division of neighbouring strings into work items (csrc/string_groups.h), compiled for the CPU with a wave of 64
lanes and compared with the rule said plainly: a group takes strings until the next one would end more than `room`
bytes after its beginning; one that ends 2^28 bytes or more after the first of its 64 is alone.  Offsets only, so
strings of any length cost nothing: a string longer than max_len may not take its neighbours' lengths away, wherever in
64 bits the text after it lies."""
import ctypes
import os
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
NOT_ENCODABLE = 0xFFF


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    out = str(tmp_path_factory.mktemp("groups") / "groups.so")
    subprocess.check_call(["g++", "-O1", "-std=c++20", "-shared", "-fPIC", "-o", out,
                           "-I", os.path.join(ROOT, "paper_2507_11941_amd", "csrc"),
                           os.path.join(ROOT, "tests", "string_groups_driver.cpp")])
    return ctypes.CDLL(out)


def groups(lib, lens, room):
    offsets = np.cumsum([0, *lens], dtype=np.int64)
    members, length = np.zeros(len(lens), np.int32), np.zeros(len(lens), np.int32)
    lib.string_groups(ctypes.c_void_p(offsets.ctypes.data), len(lens), room, ctypes.c_void_p(members.ctypes.data),
                      ctypes.c_void_p(length.ctypes.data))
    return [(int(s), int(members[s]), int(length[s])) for s in np.flatnonzero(members)]


def expected(lens, room):
    out, s = [], 0
    while s < len(lens):
        end, total = s + 1, lens[s]
        before = sum(lens[s // 64 * 64:s])
        while end < min((s // 64 + 1) * 64, len(lens)) and total + lens[end] <= room \
                and before + total + lens[end] < 2**28:
            total += lens[end]
            end += 1
        out.append((s, end - s, int(total) if total <= 1024 else NOT_ENCODABLE))
        s = end
    return out


@pytest.mark.parametrize("room", [0, 100, 1024])
@pytest.mark.parametrize("lens", [
    [0], [1024], [1025], [0] * 130, [1] * 64, [1] * 65, [512] * 63, [0, 1024, 0, 1, 0, 1023, 1025, 0, 5],
    [10, 10, 10, 300_000_000] + [20] * 70,                       # beyond 2^28 and, the next two, 2^31 and 2^32
    [10, 2**31 - 15, 5, 5, 5] + [700] * 4, [2**32 - 3, 0, 1, 2, 3] * 14, [7, 2**33, 2**40] + [30] * 130,
], ids=lambda lens: f"{len(lens)}x{lens[0]}")
def test_groups(lib, lens, room):
    assert groups(lib, lens, room) == expected(lens, room)


def test_ragged_groups(lib):
    rng = np.random.default_rng(3)
    lens = np.minimum(rng.geometric(1 / 90, size=700) - 1, 1024).tolist()
    for at in (60, 127, 128, 300):
        lens[at] = int(rng.integers(2**28, 2**34))
    for room in (60, 393, 1024):
        assert groups(lib, lens, room) == expected(lens, room)
