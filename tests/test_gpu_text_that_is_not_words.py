"""Text of which a word look-up finds little: bytes at random (most of them segments of their own), digits and letters of a
hexadecimal dump, another table's words, stretches of one letter beside single bytes (strings that are passed on out of a
group of others), in each shape of work item, without and with special tokens between the single bytes."""
import numpy as np
import pytest

import oracle
import workloads
from gpu_util import assert_same_encoding, gpu_encode

pytestmark = pytest.mark.gpu

SPECIALS = {b"<|s|>": 900001, b"\x07": 900002, b"[Q]": 900003}


def text(kind, rng, n):
    if kind == "bytes":
        return rng.integers(0, 256, size=n, dtype=np.uint8)
    if kind == "hex":
        return np.frombuffer(b"0123456789abcdef", np.uint8)[rng.integers(0, 16, size=n)]
    if kind == "few single bytes":                       # some words have none, some have two or three in 32 bytes
        data = workloads.text(3, 21, n).copy()
        data[rng.integers(0, n, size=n // 40)] = rng.integers(128, 256, size=n // 40)
        return data
    if kind == "stretches":
        data = rng.integers(0, 256, size=n, dtype=np.uint8)
        for at in rng.integers(0, n - 64, size=n // 700):
            data[at:at + 60] = 101
        return data
    return workloads.text(3, 21, n).copy()               # "other words"


@pytest.mark.parametrize("specials", [False, True])
@pytest.mark.parametrize("kind", ["bytes", "hex", "few single bytes", "stretches", "other words"])
@pytest.mark.parametrize("key", ["1k", "100k"])
def test_text(key, kind, specials):
    import torch

    assert torch.cuda.is_available(), "these tests need the GPU"
    import paper_2507_11941_amd as bpe

    rng = np.random.default_rng([len(key), len(kind), specials])
    merges = workloads.load_merges(key)
    table, own = bpe.build_table(merges), oracle.Table(merges)
    source = text(kind, rng, 3 << 20)
    if specials:
        for t in (table, own):
            t.set_specials(SPECIALS)
        for i, special in enumerate(SPECIALS):
            at = rng.integers(0, len(source) - 8, size=3000)
            source[at[:, None] + np.arange(len(special))] = np.frombuffer(special, dtype=np.uint8)
    for lens in ([300], [1024], [60001], rng.integers(0, 1025, size=900), rng.integers(0, 1025, size=3500),
                 rng.integers(0, 400, size=9000), rng.integers(0, 5000, size=600), np.minimum(rng.geometric(1 / 700, size=3000), 20000)):
        offsets = np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)
        data = source[:offsets[-1]]
        ids, off = gpu_encode(table, data, offsets)
        want_ids, want_off = own.encode_batch(data, offsets, tier=oracle.HEAP)
        assert_same_encoding(ids, off, want_ids, want_off, f"{kind}, {len(lens)} strings of up to {max(lens)}")
