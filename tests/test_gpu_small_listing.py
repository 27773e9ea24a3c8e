"""Split batches around the size up to which they are not listed (4,096 slots: strings + bytes // 896) and beyond: the most strings,
the most slots of one string each, stretches without a cut over many slots, special tokens on the nominal cut positions."""
import random

import numpy as np
import pytest

import oracle
import workloads
from gpu_util import assert_same_encoding, gpu_encode, to_batch

pytestmark = pytest.mark.gpu
TARGET, SLOTS = 896, 4096


def fill(n_strings, slots, longest):
    """Lengths of n_strings strings, one of them `longest`, with strings + bytes // 896 == slots in all."""
    left = (slots - n_strings) * TARGET + random.Random(slots).randrange(TARGET) - longest
    lens = [longest]
    for i in range(n_strings - 1):
        lens.append(min(left // (n_strings - 1 - i), 65536))
        left -= lens[-1]
    assert left <= 0 and n_strings + sum(lens) // TARGET == slots
    return lens


@pytest.mark.parametrize("specials", [False, True])
@pytest.mark.parametrize("lens", [
    [1025], [65536], [0, 0, 2000, 0], fill(4094, SLOTS, 1025), fill(4095, SLOTS + 1, 1025), fill(60, SLOTS, 65536),
    fill(1024, SLOTS, 4096), fill(1025, SLOTS - 1, 5000), fill(3000, SLOTS, 60000), fill(200, 5500, 65536),
    fill(4000, 8000, 65536), fill(9000, 9800, 3000)], ids=lambda x: f"{len(x)}x{max(x)}")
def test_small_split_batches(lens, specials):
    import torch

    assert torch.cuda.is_available(), "these tests need the GPU"
    import paper_2507_11941_amd as bpe

    merges = workloads.load_merges("1k")
    rng = np.random.default_rng(len(lens) + sum(lens))
    data = np.concatenate([workloads.text(1, 5, 2000000), np.repeat(np.frombuffer(b"et", dtype=np.uint8), 80000),
                           workloads.text(1, 6, 3000000)])[:sum(lens)].copy()
    lens = rng.permutation(lens)
    offsets = np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)
    table, own = bpe.build_table(merges), oracle.Table(merges)
    if specials:
        marks = {b"<|s|>": 5000, b"[Q]": 5001}
        table.set_specials(marks)
        own.set_specials(marks)
        for at, length in zip(offsets[:-1], lens):       # around the nominal cut positions, and at both ends
            for to in [0, length - 5, *range(TARGET - 9, int(length) - 5, TARGET)]:
                if length >= 5:
                    to = max(0, min(int(length) - 5, int(to) + int(rng.integers(0, 9))))
                    data[at + to:at + to + 5] = np.frombuffer(b"<|s|>", dtype=np.uint8)
    ids, off = gpu_encode(table, data, offsets)
    want_ids, want_off = own.encode_batch(data, offsets, tier=oracle.HEAP)
    assert_same_encoding(ids, off, want_ids, want_off, f"{len(lens)} strings")
