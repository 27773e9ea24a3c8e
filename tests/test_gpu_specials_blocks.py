"""Special tokens at the edges of the marking kernel's 16-byte chunks and 4,032-byte stretches, with strings that end inside
an occurrence, for aligned and unaligned input pointers: GPU path against the oracle."""
import random

import numpy as np
import pytest

import oracle
from gpu_util import assert_same_encoding

pytestmark = pytest.mark.gpu

SPECIALS = {b"<|endoftext|>": 70001, b"<|endoftext|>2": 70002, b"[S]": 70003, b"\x00": 70004,
            b"<" + b"q" * 62 + b">": 70005}


@pytest.mark.parametrize("shift", [0, 1, 15])
@pytest.mark.parametrize("total", [1, 15, 16, 17, 4032, 4033, 4096, 16384, 16385, 49159])
def test_marks_at_block_edges(total, shift):
    import torch

    import paper_2507_11941_amd as bpe

    rng = random.Random(total * 16 + shift)
    rows = [(97, 98), (256, 60), (124, 62), (101, 110), (113, 113)]
    text = bytearray(rng.choice(b"ab<|>[enq ") for _ in range(total))
    # occurrences that touch, cross and end at the edges
    for edge in (*range(0, total + 1, 4096), *range(4032, total + 1, 4032)):
        word = rng.choice(list(SPECIALS))
        at = edge - rng.randint(0, len(word))
        if 0 <= at and at + len(word) <= total:
            text[at:at + len(word)] = word
    cuts = sorted({0, total, *(rng.randint(0, total) for _ in range(total // 700)),
                   *(min(total, e + rng.randint(0, 70)) for e in range(0, total, 16384))})
    cuts += [total] * 2                                          # empty strings at the end
    offsets = np.array(cuts, dtype=np.int64)
    data = np.frombuffer(bytes(text), dtype=np.uint8)
    table, orc = bpe.build_table(rows), oracle.Table(rows)
    table.set_specials(SPECIALS)
    orc.set_specials(SPECIALS)
    dev = torch.device("cuda:0")
    d = torch.from_numpy(np.concatenate([np.zeros(shift, np.uint8), data])).to(dev)[shift:]
    ids, out_off = bpe.encode_batch(table, d, torch.from_numpy(offsets).to(dev), int(np.diff(offsets).max()))
    out_off = out_off.cpu().numpy()
    ids = ids[: int(out_off[-1])].cpu().numpy()
    want_ids, want_off = orc.encode_batch(data, offsets, tier=oracle.HEAP, nthreads=8)
    assert_same_encoding(ids, out_off, want_ids, want_off, f"{total} bytes, shift {shift}")
    table.free()
