"""Batches of more short strings than are resident at once: up to 4,096 strings one work item each, above that neighbours
are one item and the offsets are summed by stretches of strings.  Sizes on both sides of that line, around a workgroup's
1,024 strings and where a stretch outgrows them (131,072 strings for the list, 262,144 for the offsets); runs of empty
strings, strings at the limit, strings without a cut that go to the other encoder, and one beyond max_len (unspecified
output: with one list for all strings it yields no tokens)."""
import numpy as np
import pytest

import oracle
from gpu_util import assert_same_encoding

pytestmark = pytest.mark.gpu

ROWS = [(97, 98), (256, 99), (32, 97), (98, 98)]


@pytest.mark.parametrize("ids", ["own", "vocab", "specials"])
@pytest.mark.parametrize("batch, mean", [(1793, 200), (4096, 30), (4097, 12), (5120, 200), (8193, 500), (20011, 100), (131073, 2), (262145, 12),
                                         (300001, 1)])
def test_many_rows(batch, mean, ids):
    import torch

    import paper_2507_11941_amd as bpe

    rng = np.random.default_rng(batch)
    lens = rng.integers(0, 2 * mean + 1, size=batch)
    lens[batch // 2:batch // 2 + 700] = 0
    some = rng.permutation(batch)[:60]
    lens[some] = np.repeat([1024, 1023, 257, 256, 255, 65], 10)
    lens[some[0]], lens[0], lens[-1] = 1500, 300, 1024
    offsets = np.zeros(batch + 1, dtype=np.int64)
    np.cumsum(lens, out=offsets[1:])
    data = rng.choice(np.frombuffer(b"aabbc  x", dtype=np.uint8), size=int(offsets[-1]))
    for s in some[::3]:                                # no cut in these
        data[offsets[s]:offsets[s + 1]] = 98
    if ids != "own":
        names = rng.permutation(256 + len(ROWS)).astype(np.int32)
        args = names[:256], names[np.array(ROWS)], names[256:]
        table, orc = bpe.build_table_vocab(*args), oracle.Table(args[1], byte_ids=args[0], merged_ids=args[2])
    else:
        table, orc = bpe.build_table(ROWS), oracle.Table(ROWS)
    if ids == "specials":
        for t in (table, orc):
            t.set_specials({b"xa": 1000, b"c ": 1001})
    dev = torch.device("cuda:0")
    for max_len in (1024, 1500):                       # one list for all strings; pieces
        got, out_off = bpe.encode_batch(table, torch.from_numpy(data).to(dev), torch.from_numpy(offsets).to(dev), max_len)
        out_off = out_off.cpu().numpy()
        got = got[: int(out_off[-1])].cpu().numpy()
        want_ids, want_off = orc.encode_batch(data, offsets, tier=oracle.HEAP, nthreads=8)
        if max_len == 1024:
            at, end = want_off[some[0]], want_off[some[0] + 1]
            want_ids = np.delete(want_ids, np.s_[at:end])
            want_off = want_off - (np.arange(batch + 1) > some[0]) * (end - at)
        assert_same_encoding(got, out_off, want_ids, want_off, f"{batch} strings, max_len {max_len}")
    table.free()


def test_one_very_long_string_leaves_its_neighbours():
    """A string of 2^28 bytes among short ones, with max_len said to be 1,024: its own output is unspecified (here: no
    tokens), the strings that share its wave in the listing kernels are encoded all the same."""
    import torch

    import paper_2507_11941_amd as bpe

    rng = np.random.default_rng(28)
    lens = rng.integers(0, 60, size=5000)
    long_one, huge = 70, 1 << 28
    offsets = np.cumsum([0, *lens], dtype=np.int64)
    data = rng.choice(np.frombuffer(b"aabbc  x", dtype=np.uint8), size=int(offsets[-1]))
    dev = torch.device("cuda:0")
    at = int(offsets[long_one])
    text = torch.full((len(data) + huge,), 98, dtype=torch.uint8, device=dev)
    text[:at] = torch.from_numpy(data[:at]).to(dev)
    text[at + huge:] = torch.from_numpy(data[at:]).to(dev)
    with_long = np.concatenate([offsets[:long_one + 1], offsets[long_one:] + huge])
    table, orc = bpe.build_table(ROWS), oracle.Table(ROWS)
    got, out_off = bpe.encode_batch(table, text, torch.from_numpy(with_long).to(dev), 1024)
    out_off = out_off.cpu().numpy()
    got = got[: int(out_off[-1])].cpu().numpy()
    assert out_off[long_one + 1] == out_off[long_one]
    want_ids, want_off = orc.encode_batch(data, offsets, tier=oracle.HEAP, nthreads=8)
    assert_same_encoding(got, np.delete(out_off, long_one), want_ids, want_off, "around the long string")
    table.free()
