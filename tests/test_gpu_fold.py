"""Text that repeats itself on the GPU (csrc/fold.h): stretches of every period and around the least lengths, items of every
tier that fold, that do not (nothing repeats, too many stretches, tokens longer than what stays of a stretch), and both side
by side in a workgroup; listed and not; with special tokens in and beside the stretches; against the oracle."""
import random

import numpy as np
import pytest

import oracle
import paper_2507_11941_amd as bpe
from gpu_util import assert_same_encoding, gpu_encode, to_batch

pytestmark = pytest.mark.gpu

LENGTHS = (50, 127, 128, 129, 500, 1023, 1024, 1025, 1500, 4095, 4096, 4097, 9000, 16384, 16385, 65535, 65536)


def doubling(byte, times):
    """Rows by which a run's tokens double: longer than what stays of a stretch after five of them."""
    rows, token = [], byte
    for r in range(times):
        rows.append((token, token))
        token = 256 + r
    return rows


def random_rows(rng, rows, alphabet, n):
    rows = list(rows)
    while len(rows) < n:
        pool = list(alphabet) + [256 + r for r in range(len(rows))]
        pair = (rng.choice(pool), rng.choice(pool))
        if pair not in rows:
            rows.append(pair)
    return rows


def stretches(rng, alphabet, n):
    out = b""
    while len(out) < n:
        motif = bytes(rng.choices(alphabet, k=rng.randint(1, 9)))
        out += (motif * 2000)[:rng.choice([rng.randint(1, 20), rng.randint(16, 80), rng.randint(30, 1200), rng.randint(900, 9000)])]
    return out[:n]


def strings(rng, kind, alphabet, n):
    if kind == "runs":
        return bytes([rng.choice(alphabet)]) * n
    if kind == "periods":                                # one stretch, with a few bytes around it
        head, motif = bytes(rng.choices(alphabet, k=rng.randint(0, 30))), bytes(rng.choices(alphabet, k=rng.randint(1, 9)))
        return (head + motif * (n // len(motif)) + bytes(rng.choices(alphabet, k=rng.randint(0, 30))))[:n].ljust(n, motif[:1])
    if kind == "random":
        return bytes(rng.choices(alphabet, k=n))
    if kind == "many":                                   # more stretches than lanes, in longer text
        return b"".join(bytes([alphabet[i % len(alphabet)]]) * 60 for i in range(n // 60 + 1))[:n]
    return stretches(rng, alphabet, n)


TABLES = {
    "one byte": lambda rng: ([(97, 97)], b"ab"),
    "doubling": lambda rng: (doubling(97, 6), b"ab"),
    "tokens": lambda rng: (random_rows(rng, [], b"abc", 40), b"abc"),
    "tokens, cuts": lambda rng: (random_rows(rng, doubling(97, 2), b"abc", 30), b"abcxyz"),
}


@pytest.mark.parametrize("listed", [False, True])
@pytest.mark.parametrize("name", TABLES)
def test_texts(name, listed):
    rng = random.Random(f"{name} {listed}")
    rows, alphabet = TABLES[name](rng)
    rows = np.array(rows, np.int32)
    batch = [strings(rng, kind, alphabet, n) for kind in ("runs", "periods", "random", "many", "mixed") for n in LENGTHS]
    batch += [strings(rng, rng.choice(["periods", "mixed", "runs"]), alphabet, rng.randint(1, 3000)) for _ in range(60)]
    if listed:                                           # (more slots than are taken without a list)
        batch += [strings(rng, rng.choice(["periods", "mixed", "runs"]), alphabet, rng.randint(0, 90)) for _ in range(4000)]
    rng.shuffle(batch)
    data, offsets = to_batch(batch)
    got = gpu_encode(bpe.build_table(rows), data, offsets)
    assert_same_encoding(*got, *oracle.Table(rows).encode_batch(data, offsets, tier=oracle.HEAP), name)


@pytest.mark.parametrize("batch", [40, 5000])
def test_short_strings(batch):
    """No piece, no tier: strings of up to 1 KiB, with and without a list."""
    rng = random.Random(batch)
    rows = np.array(random_rows(rng, doubling(97, 4), b"abc", 40), np.int32)
    texts = [strings(rng, rng.choice(["runs", "periods", "mixed", "random"]), b"abc", rng.randint(0, 1024) if i % 7 else 20)
             for i in range(batch)]
    data, offsets = to_batch(texts)
    got = gpu_encode(bpe.build_table(rows), data, offsets, max_len=1024)
    assert_same_encoding(*got, *oracle.Table(rows).encode_batch(data, offsets, tier=oracle.HEAP), "rows")


@pytest.mark.parametrize("listed", [False, True])
def test_special_tokens(listed):
    """An occurrence ends a stretch, and text that is nothing but occurrences is none."""
    rng = random.Random(int(listed))
    rows = random_rows(rng, doubling(97, 3), b"abc", 30)
    specials = {b"<a>": 1000, b"aab|": 1001, b"#": 1002}
    batch = []
    for n in LENGTHS + tuple(rng.randint(96, 6000) for _ in range(40)):
        text = bytearray(strings(rng, rng.choice(["runs", "periods", "mixed"]), b"abc", n))
        for _ in range(rng.choice([0, 1, 3, 20])):
            special = rng.choice(list(specials))
            at = rng.randrange(max(1, n - 4))
            text[at:at + len(special)] = special
        batch.append(bytes(text[:n]))
    batch.append(b"<a>" * 1000)
    if listed:
        batch += [b"a" * rng.randint(0, 60) for _ in range(4200)]
    data, offsets = to_batch(batch)
    table, reference = bpe.build_table(np.array(rows, np.int32)), oracle.Table(np.array(rows, np.int32))
    table.set_specials(specials)
    reference.set_specials(specials)
    got = gpu_encode(table, data, offsets)
    assert_same_encoding(*got, *reference.encode_batch(data, offsets, tier=oracle.HEAP), "specials")


NO_CUTS = [(a, b) for a in b"ab" for b in b"ab"] + [(256, 257), (258, 256), (257, 97), (256, 256)]


def check(batch, what):
    rows = np.array(NO_CUTS, np.int32)
    data, offsets = to_batch(batch)
    got = gpu_encode(bpe.build_table(rows), data, offsets)
    assert_same_encoding(*got, *oracle.Table(rows).encode_batch(data, offsets, tier=oracle.HEAP), what)
    return len(batch) + int(offsets[-1]) // 896          # slots


@pytest.mark.parametrize("longest", [4096, 4097, 16384, 16385, 40000])
def test_workgroups_with_many_items_left(longest):
    """Batches without a list whose workgroups have several items that do not fold beside ones that do: of up to 4 KiB, to which
    four waves go, and longer ones, in LDS or not, among them."""
    rng = random.Random(longest)
    batch = [strings(rng, rng.choice(["random", "runs", "periods"]), b"ab", rng.randint(1025, 2200)) for _ in range(1200)]
    batch += [strings(rng, "random", b"ab", n) for n in (1024, 1025, 4095, 4096)]
    batch += [strings(rng, "random", b"ab", longest) for _ in range(3 if longest > 4096 else 1)]
    rng.shuffle(batch)
    assert 3000 < check(batch, "many left") <= 4096


def test_workgroup_with_items_of_all_lengths():
    """All slots of 16 neighbours in one workgroup at a time: too few for more, of every length that is treated in its own way."""
    rng = random.Random(7)
    batch = [strings(rng, "random", b"ab", n) for n in (1025, 1500, 4096, 4097, 16384, 16385, 20000, 2000, 3000, 65536)]
    assert check(batch, "all lengths") <= 256


@pytest.mark.parametrize("length, count", [(4200, 1100), (16385, 300)])
def test_long_items_that_do_not_fold(length, count):
    """More of them than there are workgroups of sixteen waves: some take a second one, by a claim (and their slab again)."""
    rng = random.Random(length)
    batch = [strings(rng, "random", b"ab", length + rng.randint(0, 700)) for _ in range(count)]
    assert check(batch, "long items") > 4096


@pytest.mark.parametrize("split", [False, True])
@pytest.mark.parametrize("longest", [150, 400])
@pytest.mark.parametrize("count", [3071, 3072, 3073, 4099, 9001])
def test_many_items_passed_on(count, longest, split):
    """Around the number from which on the last ones are claimed (four for each of 768 workgroups), and well beyond; and strings that
    are too short for that."""
    rng = random.Random(count)
    batch = [strings(rng, rng.choice(["random", "runs"]), b"ab", rng.randint(40, longest)) for _ in range(count)]
    batch += [b"a" * rng.randint(0, 20) for _ in range(1500)]
    if split:
        batch += [strings(rng, "random", b"ab", n) for n in (1025, 3000, 5000)]
    rng.shuffle(batch)
    check(batch, "passed on")
