"""Batches without strings, as a loader with a fixed max_len hands them over at the end of its data: out_offsets[0] = 0
and nothing else, for every max_len, through both entry points, the static one right after a call that left counters of
pieces in its scratch."""
import numpy as np
import pytest

import oracle
import workloads

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("specials", [False, True])
@pytest.mark.parametrize("max_len", [0, 1, 1024, 1025, 6000, 16384, 65536])
def test_no_strings(max_len, specials):
    import torch

    import paper_2507_11941_amd as bpe

    merges = workloads.load_merges("1k")
    table, orc = bpe.build_table(merges), oracle.Table(merges)
    if specials:
        for t in (table, orc):
            t.set_specials({b"<|end|>": 70001})
    dev = torch.device("cuda:0")
    nothing = torch.empty(0, dtype=torch.uint8, device=dev)
    zero = torch.zeros(1, dtype=torch.int64, device=dev)
    data, offsets = workloads.batch(1)
    offsets = offsets[[0, 20, 21, 64]]                            # strings of 5,120, 256 and 11,008 bytes
    want_ids, want_off = orc.encode_batch(data, offsets, tier=oracle.HEAP)
    d, o = torch.from_numpy(data).to(dev), torch.from_numpy(offsets).to(dev)
    workspace = torch.zeros(max(bpe.workspace_bytes(3, len(data), 11008), bpe.workspace_bytes(0, 0, max_len)),
                            dtype=torch.uint8, device=dev)

    def encode(static, data, offsets, max_len):
        ids = torch.full((max(data.numel(), 1),), -1, dtype=torch.int32, device=dev)
        off = torch.full((offsets.numel(),), -1, dtype=torch.int64, device=dev)
        if static:
            bpe.encode_batch_static(table, data, offsets, max_len, ids, off)
        else:
            bpe.encode_batch(table, data, offsets, max_len, ids, off, workspace)
        torch.cuda.synchronize()
        return ids.cpu().numpy(), off.cpu().numpy()

    for static in (False, True):
        if static and max_len > 16384:
            continue
        for _ in range(2):
            ids, off = encode(static, d, o, 11008)
            assert np.array_equal(off, want_off) and np.array_equal(ids[:off[-1]], want_ids), (static, max_len)
            ids, off = encode(static, nothing, zero, max_len)
            assert off.tolist() == [0] and ids.tolist() == [-1], (static, max_len)
    table.free()
