"""Timed cases of the encoder: what its users have it do, from one prompt to a shard of a corpus.

Every case takes a batch of strings through one of the package's encode entry points.  Shapes are those of the
benchmark's configurations, of the paper (64 to 1,024 strings of 128 to 4,096 bytes) and of everyday use around
them: a single prompt, a single long document, many short rows, ragged documents with a vocabulary's ids and
special tokens, host strings.  Texts are the synthetic word streams of ``workloads`` that belong to each table.

A case is a dict:
  api      "batch" (encode_batch, caller's buffers), "static" (encode_batch_static), "strings" (encode_strings)
  table    "1k", "32k" or "100k": the merge table, and with it the text style
  text     "words", or "motifs" (byte runs and repeated motifs), or "runs" (each string one repeated byte)
  batch    number of strings
  length   their length in bytes: all of it ("equal"), 0 to it ("uniform"), or its median ("lognormal")
  longest  upper limit of a log-normal length (else equal to length)
  mix      "equal", "uniform" or "lognormal"
  ids      "own", or "vocab": the table carries a vocabulary's ids and a set of special tokens, which the texts use
"""
from __future__ import annotations

import math
from concurrent.futures import ThreadPoolExecutor

import numpy as np
import torch

import paper_2507_11941_amd as bpe
import workloads

SPECIALS = (b"<|startoftext|>", b"<|endoftext|>", b"<|sep|>", b"[MASK]")
# bytes per token of each kind of text under its table, for work()
BYTES_PER_TOKEN = {"1k": 3.4, "32k": 6.1, "100k": 3.65, "motifs": 1.6, "runs": 1.6}


def _case(name, api, table, text, batch, length, mix="equal", longest=None, ids="own"):
    c = {"api": api, "table": table, "text": text, "batch": batch, "length": length,
         "longest": length if longest is None else longest, "mix": mix, "ids": ids}
    return dict(c, name=name) if name else c


def listed():
    return [
        # a chat turn in a serving loop: the smallest call, latency only
        _case("one prompt", "static", "32k", "words", 1, 300),
        # configuration 1: a tiny batch
        _case("64 x 256 B", "batch", "1k", "words", 64, 256),
        # a request's handful of documents, from host strings to host ids
        _case("host strings", "strings", "32k", "words", 64, 4096, "uniform"),
        # one long context
        _case("one document", "batch", "100k", "words", 1, 60001),
        # configuration 2, the middle of the paper's range
        _case("1024 x 1 KiB", "batch", "32k", "words", 1024, 1024),
        # rows of a data set: many strings of a line or two each, empty ones among them
        _case("short rows", "batch", "32k", "words", 20011, 400, "uniform"),
        # a training batch of conversations: ragged, a vocabulary's ids, special tokens
        _case("conversations", "batch", "100k", "words", 1003, 1500, "lognormal", 16384, "vocab"),
        # configuration 3: the top of the paper's string lengths in a large batch
        _case("8192 x 4 KiB", "batch", "100k", "words", 8192, 4096),
        # a corpus shard that is tokenised with a vocabulary's ids and document separators
        _case("separated documents", "batch", "100k", "words", 20000, 2048, "lognormal", 65536, "vocab"),
        # configuration 5: the benchmark's throughput workload
        _case("65536 documents", "batch", "100k", "words", 65536, 2048, "lognormal", 65536),
        # configuration 4: degenerate text (padding, separator lines, repeated markup)
        _case("runs and motifs", "batch", "100k", "motifs", 2048, 16384),
        # configuration 6: whole strings of one byte (blank or padded records), nowhere to cut
        _case("long runs", "batch", "100k", "runs", 256, 65536),
    ]


def _spread(rng, lo, hi):
    """A whole number between lo and hi, even over its logarithm."""
    return min(hi, max(lo, int(math.exp(rng.uniform(math.log(lo), math.log(hi + 1))))))


def draw(rng):
    kind = rng.choice(["prompt", "strings", "small", "small", "rows", "documents", "documents", "conversations",
                       "equal", "motifs", "runs"])
    table = rng.choice(["32k", "100k"])
    if kind == "prompt":
        return _case(None, rng.choice(["static", "batch"]), table, "words", _spread(rng, 1, 8), _spread(rng, 20, 16384))
    if kind == "strings":
        return _case(None, "strings", table, "words", _spread(rng, 1, 60), _spread(rng, 64, 16384), "uniform")
    if kind == "small":
        return _case(None, rng.choice(["static", "batch"]), rng.choice(["1k", table]), "words", _spread(rng, 16, 1024),
                     _spread(rng, 128, 4096), rng.choice(["equal", "uniform"]))
    if kind == "rows":
        return _case(None, "batch", table, "words", _spread(rng, 3000, 100000), _spread(rng, 32, 1024), "uniform",
                     ids=rng.choice(["own", "vocab"]))
    if kind == "documents":
        return _case(None, "batch", table, "words", _spread(rng, 500, 40000), _spread(rng, 512, 3000), "lognormal",
                     65536, rng.choice(["own", "vocab"]))
    if kind == "conversations":
        return _case(None, "batch", table, "words", _spread(rng, 100, 4000), _spread(rng, 300, 3000), "lognormal",
                     16384, "vocab")
    if kind == "equal":
        length = _spread(rng, 512, 16384)
        return _case(None, "batch", table, "words", _spread(rng, 1024, min(16384, (96 << 20) // length)), length)
    if kind == "motifs":
        length = _spread(rng, 1024, 65536)
        return _case(None, "batch", "100k", "motifs", _spread(rng, 16, max(16, (32 << 20) // length)), length)
    return _case(None, "batch", "100k", "runs", _spread(rng, 16, 400), _spread(rng, 8192, 65536))


def _words(style, seed, nbytes):
    """A word stream of nbytes, in up to sixteen stretches made side by side."""
    part = max(1 << 20, -(-nbytes // 16))
    sizes = [min(part, nbytes - at) for at in range(0, nbytes, part)]
    workloads.text(style, 0, 1)                        # the style's word list exists before the threads start
    with ThreadPoolExecutor(len(sizes) or 1) as pool:
        parts = list(pool.map(lambda i: workloads.text(style, 1000 * seed + i, sizes[i]), range(len(sizes))))
    return parts[0] if len(parts) == 1 else np.concatenate(parts or [np.empty(0, np.uint8)])


def _lengths(case, rng):
    """The strings' lengths: the case says which, the seed in which order (so that all seeds have equal totals)."""
    n, length = case["batch"], case["length"]
    own = np.random.default_rng((n, length, case["longest"]))
    if case["mix"] == "uniform":
        lens = own.integers(0, length + 1, size=n)
        lens[0] = length
    elif case["mix"] == "lognormal":
        lens = np.clip(np.rint(length * np.exp(own.standard_normal(n))), 16, case["longest"])
    else:
        lens = np.full(n, length)
    return rng.permutation(lens.astype(np.int64))


def _mark(data, offsets, rng):
    """Specials into the text: the first and last bytes of most strings, and one at about every 600th byte."""
    begin, end = offsets[:-1], offsets[1:]
    roomy = (end - begin) >= 64

    def put(at, text):
        data[at[:, None] + np.arange(len(text))] = np.frombuffer(text, dtype=np.uint8)

    put(begin[roomy], SPECIALS[0])
    put(end[roomy] - len(SPECIALS[1]), SPECIALS[1])
    if len(data) > 64:
        put(rng.integers(0, len(data) - 16, size=len(data) // 1200), SPECIALS[2])
        put(rng.integers(0, len(data) - 16, size=len(data) // 1200), SPECIALS[3])


def prepare(case, seed):
    rng = np.random.default_rng(seed)
    merges = workloads.load_merges(case["table"])
    if case["ids"] == "vocab":
        names = rng.permutation(256 + len(merges)).astype(np.int32)
        own = merges.astype(np.int64)
        table = bpe.build_table_vocab(names[:256], names[own], names[256:])
        table.set_specials({text: 256 + len(merges) + i for i, text in enumerate(SPECIALS)})
    else:
        table = bpe.build_table(merges)

    lens = _lengths(case, rng)
    offsets = np.zeros(len(lens) + 1, dtype=np.int64)
    np.cumsum(lens, out=offsets[1:])
    total, longest = int(offsets[-1]), int(lens.max())
    if case["text"] == "runs":
        data = np.repeat(rng.choice(np.frombuffer(b"a0 e", dtype=np.uint8), size=len(lens)), lens)
    elif case["text"] == "motifs":
        data = workloads.adversarial(seed, case["batch"], case["length"])
    else:
        data = _words({"1k": 1, "32k": 2, "100k": 3}[case["table"]], seed, total)
    if case["ids"] == "vocab":
        _mark(data, offsets, rng)

    if case["api"] == "strings":
        raw = data.tobytes()
        return {"api": "strings", "table": table, "flat": np.zeros(total, dtype=np.int32),
                "strings": [raw[offsets[i]:offsets[i + 1]] for i in range(len(lens))]}
    dev = torch.device("cuda:0")
    state = {"api": case["api"], "table": table, "max_len": longest,
             "data": torch.from_numpy(data).to(dev), "offsets": torch.from_numpy(offsets).to(dev),
             # (zeroed, so that the part of the ids buffer that an encoding does not reach has a value too)
             "ids": torch.zeros(max(total, 1), dtype=torch.int32, device=dev),
             "out_offsets": torch.zeros(len(lens) + 1, dtype=torch.int64, device=dev)}
    if case["api"] == "batch":
        state["workspace"] = torch.empty(bpe.workspace_bytes(len(lens), total, longest), dtype=torch.uint8, device=dev)
    return state


def run(state):
    if state["api"] == "strings":
        rows = bpe.encode_strings(state["table"], state["strings"])
        counts = np.fromiter(map(len, rows), dtype=np.int64, count=len(rows))
        np.concatenate(rows, out=state["flat"][:counts.sum()])       # into the batch's one buffer, as a loader does
        return state["flat"], counts
    if state["api"] == "static":
        return bpe.encode_batch_static(state["table"], state["data"], state["offsets"], state["max_len"], state["ids"],
                                       state["out_offsets"])
    return bpe.encode_batch(state["table"], state["data"], state["offsets"], state["max_len"], state["ids"],
                            state["out_offsets"], state["workspace"])


def work(case):
    """Each byte read once, each id written once (4 bytes), one offset per string read and one written."""
    mean = {"equal": 1.0, "uniform": 0.5, "lognormal": math.exp(0.5)}[case["mix"]] * case["length"]
    nbytes = case["batch"] * min(mean, case["longest"])
    kind = case["text"] if case["text"] != "words" else case["table"]
    return {"bytes": nbytes + 4.0 * nbytes / BYTES_PER_TOKEN[kind] + 16.0 * (case["batch"] + 1), "flops": 0.0}


def tolerance(case):
    return "exact"                                     # ids and offsets are whole numbers
