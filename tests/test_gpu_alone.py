"""A batch of one string of up to 1 KiB, which one kernel encodes into the output: plain, with a vocabulary's ids, with special
tokens, with a segment of more than 32 bytes (another encoder's), empty; through both entry points."""
import numpy as np
import pytest

import oracle
import workloads
from gpu_util import assert_same_encoding, gpu_encode

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("ids", ["own", "vocab"])
@pytest.mark.parametrize("text", ["words", "specials", "run"])
@pytest.mark.parametrize("length", [0, 1, 2, 33, 300, 1023, 1024])
def test_one_string(length, text, ids):
    import torch

    assert torch.cuda.is_available(), "these tests need the GPU"
    import paper_2507_11941_amd as bpe

    merges = workloads.load_merges("1k")
    rng = np.random.default_rng(length)
    names = rng.permutation(256 + len(merges)).astype(np.int32)
    if ids == "vocab":
        args = names[:256], names[merges], names[256:]
        table, own = bpe.build_table_vocab(*args), oracle.Table(args[1], args[0], args[2])
    else:
        table, own = bpe.build_table(merges), oracle.Table(merges)
    data = workloads.text(1, 9, 4096)[:length].copy()
    if text == "run":
        data[:length // 2] = ord("e")
    elif text == "specials":
        for t in (table, own):
            t.set_specials({b"<s>": 7000})
        for at in (0, length // 2, length - 3):
            if length >= 12:
                data[at:at + 3] = np.frombuffer(b"<s>", dtype=np.uint8)
    offsets = np.array([0, length], dtype=np.int64)
    want_ids, want_off = own.encode_batch(data, offsets)
    got_ids, got_off = gpu_encode(table, data, offsets)
    assert_same_encoding(got_ids, got_off, want_ids, want_off, "with a workspace")
    dev = torch.device("cuda:0")
    d = torch.from_numpy(data).to(dev) if length else torch.empty(0, dtype=torch.uint8, device=dev)
    out, off = torch.empty(max(length, 1), dtype=torch.int32, device=dev), torch.empty(2, dtype=torch.int64, device=dev)
    for _ in range(3):
        out.fill_(-1)
        off.fill_(-1)
        bpe.encode_batch_static(table, d, torch.from_numpy(offsets).to(dev), length, out, off)
        torch.cuda.synchronize()
        got_off = off.cpu().numpy()
        assert_same_encoding(out.cpu().numpy()[:got_off[1]], got_off, want_ids, want_off, "static")


@pytest.mark.parametrize("ids", ["own", "vocab"])
@pytest.mark.parametrize("batch", [1, 2, 3073])
@pytest.mark.parametrize("max_len", [0, 300, 1024, 1025])
def test_empty_strings_without_an_ids_buffer(max_len, batch, ids):
    """A tensor without elements has a null pointer, which is a valid out_ids where there are no bytes."""
    import torch

    assert torch.cuda.is_available(), "these tests need the GPU"
    import paper_2507_11941_amd as bpe

    merges = workloads.load_merges("1k")
    names = np.random.default_rng(1).permutation(256 + len(merges)).astype(np.int32)
    table = bpe.build_table(merges) if ids == "own" else bpe.build_table_vocab(names[:256], names[merges], names[256:])
    dev = torch.device("cuda:0")
    data, out = torch.empty(0, dtype=torch.uint8, device=dev), torch.empty(0, dtype=torch.int32, device=dev)
    assert out.data_ptr() == 0
    offsets = torch.zeros(batch + 1, dtype=torch.int64, device=dev)
    for encode in (bpe.encode_batch, bpe.encode_batch_static):
        off = torch.full((batch + 1,), -1, dtype=torch.int64, device=dev)
        encode(table, data, offsets, max_len, out, off)
        torch.cuda.synchronize()
        assert not off.any().item(), encode.__name__
