"""The table of whole words (csrc/word_table.h), compiled for the CPU: a token of 2 to 15 bytes is taken in only when
Algorithm 1 turns its bytes into that token (the oracle says), nearly all of those are, what is found is the oracle's encoding, and nothing else
is found."""
import ctypes
import os
import random
import subprocess

import numpy as np
import pytest

import oracle
import paper_2507_11941_amd as bpe
import workloads

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
WORD_BYTES = 15


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    out = str(tmp_path_factory.mktemp("words") / "words.so")
    subprocess.check_call(["g++", "-O1", "-std=c++17", "-shared", "-fPIC", "-o", out,
                           "-I", os.path.join(ROOT, "paper_2507_11941_amd", "csrc"),
                           os.path.join(ROOT, "tests", "word_table_driver.cpp")])
    return ctypes.CDLL(out)


def ptr(a):
    return ctypes.c_void_p(a.ctypes.data)


def chained_table(rng, n_rows, alphabet):
    """Random rows, biased towards recent tokens; many of their tokens do not encode to themselves."""
    rows, seen = [], set()
    while len(rows) < n_rows:
        pool = list(alphabet) + [256 + r for r in range(len(rows))]
        a = rng.choice(pool) if rng.random() < 0.6 else rng.choice(pool[-20:])
        b = rng.choice(pool) if rng.random() < 0.6 else rng.choice(pool[-20:])
        if (a, b) not in seen:
            seen.add((a, b))
            rows.append((a, b))
    return np.array(rows, dtype=np.int32).reshape(-1, 2)


def check(lib, merges, rng, others):
    merges = np.ascontiguousarray(merges, dtype=np.int32).reshape(-1, 2)
    n = len(merges)
    image, log2_image = bpe.table_image(merges)
    built = []
    for words_image in (None, image):                    # ranks from a map, and from the table as the library has them
        known, keys = np.zeros(256 + n, np.uint8), np.zeros((256 + n) * 4, np.uint32)
        buckets = np.zeros(1 << 20, np.uint32)
        log2 = lib.build_words(ptr(merges), n, None if words_image is None else ptr(words_image), log2_image, ptr(known),
                               ptr(buckets), ctypes.c_int64(len(buckets)), ptr(keys))
        assert log2 >= 0
        built.append((log2, known, buckets, keys))
    assert all(np.array_equal(a, b) for a, b in zip(*built))
    expansion = [bytes([b]) for b in range(256)]
    for a, b in merges.tolist():
        expansion.append((expansion[a] + expansion[b])[:WORD_BYTES + 1])      # (a long one stays long)
    words = [t for t in range(256, 256 + n) if len(expansion[t]) <= WORD_BYTES]
    strings = [expansion[t] for t in words] + others
    data = np.frombuffer(b"".join(strings), dtype=np.uint8).copy()
    offsets = np.cumsum([0] + [len(x) for x in strings], dtype=np.int64)
    ids, off = oracle.Table(merges).encode_batch(data, offsets, tier=oracle.TEXTBOOK)

    def find(text):
        raw = np.frombuffer(text, dtype=np.uint8).copy()
        return lib.find_word(ptr(buckets), log2, ptr(keys), ptr(raw), len(raw))

    missing = 0
    for i, t in enumerate(words):
        single = off[i + 1] - off[i] == 1 and ids[off[i]] == t
        assert single or not known[t], (t, expansion[t])
        got = find(expansion[t])
        if got < 0:
            missing += single
        else:
            assert off[i + 1] - off[i] == 1 and ids[off[i]] == got
    for t in range(256, 256 + n):
        assert len(expansion[t]) <= WORD_BYTES or not known[t]
    for i, text in enumerate(others, start=len(words)):
        got = find(text)
        if off[i + 1] - off[i] != 1:
            assert got == -1, text
        else:
            assert got in (-1, ids[off[i]])
    return missing, int(known[256:].sum())


@pytest.mark.parametrize("seed", range(6))
def test_random_tables(lib, seed):
    rng = random.Random(seed)
    for _ in range(25):
        alphabet = rng.sample(range(256), rng.choice([1, 2, 3, 8, 60])) + [0]
        merges = chained_table(rng, rng.choice([0, 1, 5, 40, 300]), alphabet)
        others = [bytes(rng.choices(alphabet, k=rng.randint(2, WORD_BYTES))) for _ in range(100)]
        missing, known = check(lib, merges, rng, others)
        assert missing <= 3 + known // 20


@pytest.mark.parametrize("table,style", [("1k", 1), ("32k", 2), ("100k", 3)])
def test_trained_tables(lib, table, style):
    text = workloads.text(style, 77, 40000).tobytes()
    others = [text[i:i + 2 + i % (WORD_BYTES - 1)] for i in range(0, 30000, 17)]
    missing, known = check(lib, workloads.load_merges(table), random.Random(1), others)
    assert known > 0 and missing <= known // 30            # full buckets: one word in sixty


@pytest.mark.parametrize("table", ["1k", "32k", "100k"])
def test_ranks_in_a_table_image(lib, table):
    """Every row is found at its rank, those outside their home bucket too, and no other pair is found."""
    lib.rank_in_image.restype = ctypes.c_int64
    merges = workloads.load_merges(table)
    image, log2 = bpe.table_image(merges)
    tags = image[:4 << log2][1::2]
    if table != "1k":
        assert ((tags != 0xFFFFFFFF) & (tags >> 28 != 0)).any()        # displaced rows
    for r, (a, b) in enumerate(merges.tolist()):
        assert lib.rank_in_image(ptr(image), log2, a, b) == r
    rows = set(map(tuple, merges.tolist()))
    rng, lefts = random.Random(len(rows)), merges[:, 0].tolist()
    for _ in range(50000):
        a, b = lefts[rng.randrange(len(lefts))], rng.randrange(256 + len(merges))
        if (a, b) not in rows:
            assert lib.rank_in_image(ptr(image), log2, a, b) == -1
