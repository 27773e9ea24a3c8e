"""Whole-word look-ups and what they leave to the merges: segments that are one token, that are not, and that no key holds
(16 bytes and more), at the edges of the kernel's lists -- more segments than are listed at a time, more of them to be
merged than the arena or the job list takes (several rounds over one item), single bytes only, texts that end within the
last wide load -- in each shape of work item: strings without a work list, short items, long items of pieces or strings."""
import random

import numpy as np
import pytest

import oracle
from gpu_util import assert_same_encoding, gpu_encode, to_batch

pytestmark = pytest.mark.gpu

CUT = b"\x00\x01\x02\x03"                                # bytes of no row


def table(rng):
    """Rows over eight letters, many of whose tokens do not encode to themselves, and a row whose junction ("a", "d") is
    no pair itself: "ad" is a segment of two bytes that no row joins."""
    letters = list(b"abcdefgh")
    rows = [(97, 98), (100, 101), (256, 97), (100, 257), (258, 259)]     # ab, de, aba, dde, aba+dde
    seen = set(rows)
    while len(rows) < 400:
        pool = letters + [256 + r for r in range(len(rows))]
        p = (rng.choice(pool), rng.choice(pool if rng.random() < 0.5 else letters))
        if p not in seen and p != (97, 100):
            seen.add(p)
            rows.append(p)
    return np.array(rows, dtype=np.int32)


def words(rng, kind, merges):
    tokens = [bytes([b]) for b in range(256)]
    for a, b in merges.tolist():
        tokens.append((tokens[a] + tokens[b])[:40])
    if kind == "bytes":
        return [bytes([c]) for c in CUT]
    if kind == "pairs":                                  # 341 jobs a KiB: more than a list of jobs
        return [b"ad"]
    if kind == "tokens":
        return [t for t in tokens[256:] if len(t) <= 15]
    if kind == "keys":                                   # on both sides of a key's length and of a lane's
        return [bytes(rng.choices(b"abcdefgh", k=n)) for n in (2, 3, 14, 15, 16, 17, 31, 32) for _ in range(20)]
    if kind == "long":                                   # more bytes to merge than the arena holds
        return [bytes(rng.choices(b"abcdefgh", k=n)) for n in (29, 30, 31, 32) for _ in range(20)]
    return [bytes(rng.choices(b"abcdefgh", k=rng.choice([1, 2, 3, 5, 8, 13]))) for _ in range(200)] + \
        ([bytes(rng.choices(b"abcdefgh", k=40))] if kind == "mixed" else [])


def text(rng, vocabulary, length):
    out = []
    size = 0
    while size < length:
        out.append(rng.choice(vocabulary))
        out.append(bytes([rng.choice(CUT)]))
        size += len(out[-2]) + 1
    return b"".join(out)[:length]


@pytest.mark.parametrize("kind", ["bytes", "pairs", "tokens", "keys", "long", "short", "mixed"])
@pytest.mark.parametrize("shape", ["direct", "pieces", "long pieces", "strings", "long strings"])
def test_words(shape, kind):
    import torch

    assert torch.cuda.is_available(), "these tests need the GPU"
    import paper_2507_11941_amd as bpe

    rng = random.Random(shape + kind)
    merges = table(rng)
    vocabulary = words(rng, kind, merges)
    source = text(rng, vocabulary, 300000)

    def string(n):
        at = rng.randrange(len(source) - n)
        return source[at:at + n]

    batches = {
        "direct": [[string(n)] for n in (1, 2, 15, 16, 17, 1023, 1024)] + [[string(rng.randint(0, 1024)) for _ in range(90)]],
        "pieces": [[string(n) for n in (1025, 2047, 2048, 2049, 4095, 60001)], [string(rng.randint(0, 5000)) for _ in range(300)]],
        "long pieces": [[string(rng.choice([0, 3, 900, 1800, 4096, 5000])) for _ in range(2500)]],
        "strings": [[string(rng.randint(0, 1024)) for _ in range(3500)]],
        "long strings": [[string(rng.randint(0, 900)) for _ in range(9000)]],
    }[shape]
    t, o = bpe.build_table(merges), oracle.Table(merges)
    for strings in batches:
        data, offsets = to_batch(strings)
        ids, off = gpu_encode(t, data, offsets)
        want_ids, want_off = o.encode_batch(data, offsets, tier=oracle.HEAP)
        assert_same_encoding(ids, off, want_ids, want_off, f"{shape}, {kind}, {len(strings)} strings")


@pytest.mark.parametrize("n_bytes", [0, 1, 96, 97, 5000, 300000])
def test_host_strings_of_a_token_a_byte(n_bytes):
    """More tokens than are fetched at first (a third of the bytes, and 64)."""
    import paper_2507_11941_amd as bpe

    rng = np.random.default_rng(n_bytes)
    data = rng.integers(0, 256, size=n_bytes, dtype=np.uint8).tobytes()
    strings = [data[i:i + 777] for i in range(0, n_bytes, 777)] + [b"", "aé"]
    got = bpe.encode_strings(bpe.build_table([]), strings)
    assert [x.dtype for x in got] == [np.int32] * len(strings)
    assert [x.tolist() for x in got] == [list(s if isinstance(s, bytes) else s.encode()) for s in strings]
