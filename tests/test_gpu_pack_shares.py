"""Pieces that run over void slots, whose ids are copied in shares by those slots: strings without a cut and without a
merge (one id per byte, the most a piece can have), around the share size and up to the longest string, alone and
among enough short strings that the kernels for large batches run; plain and vocabulary ids."""
import numpy as np
import pytest

import oracle
from gpu_util import assert_same_encoding

pytestmark = pytest.mark.gpu

# (b, c) and (c, b) lie at junctions of the last two rows but are no rows: "bcbc..." has no cut and never merges
ROWS = [(97, 98), (98, 97), (256, 99), (99, 257)]
LENGTHS = [1025, 1792, 1793, 2047, 4096, 4097, 16385, 65536]


@pytest.mark.parametrize("vocab", [False, True])
@pytest.mark.parametrize("short_rows", [0, 5000])
def test_long_pieces(short_rows, vocab):
    import torch

    import paper_2507_11941_amd as bpe

    rows = [b"bc" * (n // 2) + b"b" * (n % 2) for n in LENGTHS]
    rows += [b"bc" * 600 + b" " + b"cb" * 700, b"ab" * 4000 + b"bc" * 3000, b"", b" "]
    rows += [b"ab cb"[: i % 6] for i in range(short_rows)]
    order = np.random.default_rng(short_rows).permutation(len(rows))
    rows = [rows[i] for i in order]
    offsets = np.cumsum([0] + [len(r) for r in rows]).astype(np.int64)
    data = np.frombuffer(b"".join(rows), dtype=np.uint8)
    if vocab:
        names = np.random.default_rng(1).permutation(260).astype(np.int32)
        args = names[:256], names[np.array(ROWS)], names[256:]
        table, orc = bpe.build_table_vocab(*args), oracle.Table(args[1], byte_ids=args[0], merged_ids=args[2])
    else:
        table, orc = bpe.build_table(ROWS), oracle.Table(ROWS)
    dev = torch.device("cuda:0")
    ids, out_off = bpe.encode_batch(table, torch.from_numpy(data.copy()).to(dev), torch.from_numpy(offsets).to(dev),
                                    max(LENGTHS))
    out_off = out_off.cpu().numpy()
    ids = ids[: int(out_off[-1])].cpu().numpy()
    want_ids, want_off = orc.encode_batch(data, offsets, tier=oracle.HEAP, nthreads=8)
    assert_same_encoding(ids, out_off, want_ids, want_off, f"{short_rows} short rows")
    table.free()
