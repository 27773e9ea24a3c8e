"""Folding (csrc/fold.h), compiled for the CPU with a wave of 64 lanes: what is left out repeats what stays, and the encoding
of what stays (by the oracle), with each stretch's block put back in as often as it was left out, is the encoding of the
whole text -- for text of runs and motifs over random tables, in which tokens join in every way, and over a trained one."""
import ctypes
import os
import subprocess

import numpy as np
import pytest

import oracle
import workloads

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HISTORY, MOST = 24, 1024


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    out = str(tmp_path_factory.mktemp("fold") / "fold.so")
    subprocess.check_call(["g++", "-O1", "-std=c++20", "-shared", "-fPIC", "-o", out,
                           "-I", os.path.join(ROOT, "paper_2507_11941_amd", "csrc"),
                           os.path.join(ROOT, "tests", "fold_driver.cpp")])
    return ctypes.CDLL(out)


def fold(lib, data, marks=None, most=MOST):
    """(stretches [k, 5], bytes that stay), or None."""
    def padded(a):
        return None if a is None else np.concatenate([a, np.zeros(16, np.uint8)])
    text, mark = padded(data), padded(marks)
    out, stay = np.zeros((64, 5), np.uint32), ctypes.c_int(0)
    k = lib.fold(ctypes.c_void_p(text.ctypes.data), ctypes.c_void_p(None if mark is None else mark.ctypes.data), len(data), most,
                 ctypes.c_void_p(out.ctypes.data), ctypes.byref(stay))
    return None if k < 0 else (out[:k].astype(np.int64), stay.value)


def kept(data, stretches, marks=None):
    """Which bytes stay; every stretch repeats itself as it claims, and holds no mark."""
    keep, left_out, last = np.ones(len(data), bool), 0, -18
    for x, out, q, first, end in stretches.tolist():
        raw = x + left_out
        whole = np.arange(raw - (HISTORY - 1), raw + out + (end - x))
        assert 1 <= q <= 8 and first == x - (HISTORY - 1) - q and x - last >= 18 and raw - (HISTORY - 1) - q >= 0
        assert (data[whole] == data[whole - q]).all()
        if marks is not None:
            assert not marks[whole].any() and not marks[whole - q].any()
        keep[raw:raw + out] = False
        left_out += out
        last = x
    return keep


def encode(table, data):
    return table.encode_batch(data, np.array([0, len(data)]), tier=oracle.TEXTBOOK)[0]


def encode_folded(lib, table, size_of, data):
    """The ids by way of the folded text; None if it does not fold or some stretch has no block."""
    folded = fold(lib, data)
    if folded is None:
        return None
    stretches, stay = folded
    text = data[kept(data, stretches)]
    assert len(text) == stay
    ids = encode(table, text)
    starts = np.concatenate([[0], np.cumsum(size_of[ids])])
    is_start = np.zeros(len(text) + 80, bool)
    is_start[starts] = True
    out, done, end_before = [], 0, 0
    for x, left_out, q, first, end in stretches.tolist():
        if left_out:
            w = sum(1 << i for i in range(64) if is_start[first + i])
            found = (ctypes.c_uint32 * 2)()
            lib.block(ctypes.c_uint64(w), end - first, q, max(end_before - first, 0), found)
            at, size = first + found[0], found[1]
            if size == 0:
                return None
            assert left_out % size == 0 and size % q == 0 and at + 2 * size <= end
            i, j = np.searchsorted(starts, [at + size, at + 2 * size])
            assert np.array_equal(ids[i:j], ids[2 * i - j:i]) and done <= 2 * i - j
            out += [ids[done:j], np.tile(ids[i:j], left_out // size)]
            done = j
        end_before = end
    return np.concatenate(out + [ids[done:]])


def stretch_text(rng, alphabet, n):
    parts, total = [], 0
    while total < n:
        motif = rng.choice(alphabet, size=rng.integers(1, 10))
        size = [rng.integers(1, 20), rng.integers(16, 80), rng.integers(30, 1200), rng.integers(1000, 5000)]
        length = int(min(n - total, size[rng.choice(4, p=[.35, .3, .3, .05])]))
        parts.append(np.resize(motif, length))
        total += length
    return np.concatenate(parts).astype(np.uint8)


def random_table(rng, alphabet, rows):
    merges, pool = [], list(map(int, alphabet))
    for _ in range(20 * rows):
        pair = (pool[rng.integers(len(pool))], pool[rng.integers(len(pool))])
        if len(merges) < rows and pair not in merges:
            merges.append(pair)
            pool.append(255 + len(merges))
    return np.array(merges, np.int32)


def token_sizes(merges):
    size = np.ones(256 + len(merges), int)
    for r, (a, b) in enumerate(merges):
        size[256 + r] = size[a] + size[b]
    return size


def test_random_tables(lib):
    rng = np.random.default_rng(1)
    done = 0
    for _ in range(40):
        alphabet = np.arange(97, 97 + rng.integers(1, 5))
        merges = random_table(rng, alphabet, int(rng.integers(1, 40)))
        data = stretch_text(rng, alphabet, int(rng.integers(96, 5000)))
        table = oracle.Table(merges)
        got = encode_folded(lib, table, token_sizes(merges), data)
        if got is not None:
            done += 1
            assert np.array_equal(got, encode(table, data))
    assert done >= 25


def test_trained_table(lib):
    merges = workloads.load_merges("100k")
    table, sizes = oracle.Table(merges), token_sizes(merges)
    for seed, n in enumerate((96, 200, 1023, 1024, 1025, 2048, 4000, 8192)):
        data = workloads.adversarial(100 + seed, 1, n)
        got = encode_folded(lib, table, sizes, data)
        assert got is not None and np.array_equal(got, encode(table, data))


@pytest.mark.parametrize("q", range(1, 10))
def test_one_stretch(lib, q):
    """Around the least lengths, the ends of rows and whole rows; a period of nine is none."""
    rng = np.random.default_rng(q)
    motif = np.arange(97, 97 + q)
    for n in [96, 1023, 1024, 1025, 4096, 5000, 65536] + [int(v) for v in rng.integers(96, 3000, 6)]:
        for before in (0, 1, 15, 40) if n < 5000 else (q,):
            data = np.concatenate([np.arange(before) + 160, np.resize(motif, n - before)]).astype(np.uint8)
            folded = fold(lib, data, most=100000)
            keep = kept(data, folded[0])
            assert keep.sum() == folded[1]
            unit = 8 if q <= 2 else 2 * q
            if q <= 8:                                   # the text's first eight bytes count as no repetition
                start = max(before + q, 8)
                assert folded[1] == start + HISTORY - 1 + (n - start - (HISTORY - 1)) % unit
            else:
                assert folded[1] == n


@pytest.mark.parametrize("q", range(1, 9))
def test_least_stretches(lib, q):
    """A stretch that is just long enough is found wherever it lies, in text that is short, of two rows, and beyond them."""
    rng = np.random.default_rng(10 + q)
    unit = 8 if q <= 2 else 2 * q
    for n in (128, 1024, 1040, 2048, 2100):
        for at in (*range(8, 25), n - 16 - q - HISTORY - unit, *(int(v) for v in rng.integers(8, n - 60, 4))):
            data = rng.permutation(np.resize(np.arange(100, 256), n)).astype(np.uint8)
            size = q + HISTORY - 1 + unit
            data[at:at + size] = np.resize(np.arange(1, q + 1), size)
            stretches, stay = fold(lib, data, most=100000)
            assert len(stretches) == 1 and stay == n - unit and stretches[0][0] == at + q + HISTORY - 1


def emission_texts():
    """(name, merges, text): stretches of few and many copies, of ids that fill whole stores or not, at all places of the lanes' columns."""
    rng = np.random.default_rng(6)
    trained = workloads.load_merges("100k")
    for seed, n in enumerate((128, 500, 1024, 1500, 4000, 16384, 65536)):
        yield "trained", trained, workloads.adversarial(200 + seed, 1, n)
    for _ in range(120):
        alphabet = np.arange(97, 97 + rng.integers(1, 5))
        yield "random", random_table(rng, alphabet, int(rng.integers(1, 40))), stretch_text(rng, alphabet, int(rng.integers(128, 9000)))
    pairs = np.array([(97, 98), (256, 97)], np.int32)
    for q in range(1, 9):                                # copies of 1,000 to 1,100 ids, and of 65,000
        motif = np.arange(97, 97 + q)
        for n in (1000 + 24 + 2 * q, 1024 + 24 + q, 1100, 1300, 65536):
            yield "one stretch", pairs, np.concatenate([np.arange(q) + 160, np.resize(motif, n)])[:65536].astype(np.uint8)
    for size in range(16, 1009, 31):                     # what stays: one byte a lane to sixteen
        words = rng.permutation(np.resize(np.arange(100, 256), size))
        yield "what stays", pairs, np.concatenate([words, np.resize([97, 98, 97], 400)]).astype(np.uint8)


def test_emission(lib, tmp_path):
    """The ids that emit_folded() writes, from the oracle's tokens of what stays, in buffers of just the size they must have, with the
    address and undefined-behaviour sanitizers looking on."""
    exe = str(tmp_path / "fold")
    subprocess.check_call(["g++", "-O1", "-g", "-std=c++20", "-DFOLD_PROGRAM", "-fsanitize=address,undefined", "-fno-sanitize-recover=all",
                           "-static-libasan", "-o", exe, "-I", os.path.join(ROOT, "paper_2507_11941_amd", "csrc"),
                           os.path.join(ROOT, "tests", "fold_driver.cpp")])
    records, want = [], []
    for name, merges, data in emission_texts():
        table, sizes = oracle.Table(merges), token_sizes(merges)
        folded = fold(lib, data)
        if folded is None or len(folded[0]) == 0:
            continue
        ids = encode(table, data[kept(data, folded[0])])
        whole = encode(table, data)
        want.append((name, whole, encode_folded(lib, table, sizes, data)))
        records.append(np.array([len(data), len(ids), len(whole)], np.int32).tobytes() + data.tobytes() +
                       sizes[ids].astype(np.int32).tobytes() + ids.astype(np.int32).tobytes())
    run = subprocess.run([exe], input=b"".join(records), capture_output=True, timeout=120,
                         env=dict(os.environ, ASAN_OPTIONS="verify_asan_link_order=0:detect_stack_use_after_return=0"))
    assert run.returncode == 0, run.stderr[-2000:].decode()
    got, done = np.frombuffer(run.stdout, np.int32), 0
    for name, whole, model in want:
        k = int(got[0])
        if model is None:                                # a stretch without a block: nothing is written
            assert k == -1, name
        else:
            done += 1
            assert np.array_equal(got[1:1 + k], whole), name
        got = got[1 + max(k, 0):]
    assert done >= 100 and len(got) == 0


def test_marks(lib):
    rng = np.random.default_rng(3)
    for _ in range(40):
        data = stretch_text(rng, np.arange(97, 100), int(rng.integers(96, 4000)))
        marks = (rng.random(len(data)) < 1 / 300).astype(np.uint8)
        folded = fold(lib, data, marks, most=100000)
        if folded is not None:
            kept(data, folded[0], marks)


def test_too_much_stays(lib):
    rng = np.random.default_rng(4)
    words = rng.integers(0, 256, 5000).astype(np.uint8)
    assert fold(lib, words) is None                      # nothing repeats
    many = np.concatenate([np.resize([97 + i % 5], 60) for i in range(70)]).astype(np.uint8)
    assert fold(lib, many, most=100000) is None          # more than 64 stretches
    assert fold(lib, many[:64 * 60], most=100000) is not None
