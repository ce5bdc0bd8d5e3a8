"""Performance cases of the QLC codec: what programs call it for, over the range they call it on.

A case names an operation, a symbol count n (for the batched operations: the number of tensors and the
range of their sizes), a chunk size, an alphabet, a layout mode and the distribution of the values:

  compress      qlc_compress / qlc_compress_sym: histogram, table and encode of one tensor
  encode        qlc_encode / qlc_encode_sym: encode with a table built beforehand from another tensor of
                the same type (one table per tensor type, fixed in advance)
  decode        qlc_decode / qlc_decode_sym: the automatic choice of decoder
  table         qlc_build_table: histogram and table only (calibrating a tensor type)
  batch_encode  qlc_encode_batched: many uneven tensors in one call
  batch_decode  qlc_decode_batched

A program keeps its buffers and its workspace from call to call, so they belong to the state.  Bitstream
buffers start out as zeros: past the end of the stream nothing is written, and the whole buffer is returned.
"""
import math
import random

import torch

from paper_2602_17849_amd import datagen, qlc

# Bits per symbol that each distribution codes to under its searched table, for work().
CODE_BITS = {"gaussian": 6.70, "laplace": 7.01, "student_t": 6.75, "weights": 6.70, "uniform": 8.0,
             "zeros90": 3.40, "e3m2": 4.64, "e2m1": 3.65}

MODES = {"quad": qlc.LAYOUT_SEARCH_QUAD, "any": qlc.LAYOUT_SEARCH_ANY, "paper_t1": qlc.LAYOUT_PAPER_T1,
         "m64a8": qlc.LAYOUT_M64_AREAS8, "m16a4": qlc.LAYOUT_M16_AREAS4}

SMALLEST, LARGEST = 1 << 16, 1 << 28
BATCH_LO, BATCH_HI = 1 << 20, 32 << 20     # one shard of the 1152-shard batch
BATCH_MAX_TENSORS = 64


def listed():
    return [
        # the smallest requests the serving loop takes (64 KiB at C = 512): launches and latency
        {"name": "compress_64k", "op": "compress", "n": 1 << 16, "chunk": 512, "bits": 8, "mode": "quad", "data": "laplace"},
        {"name": "decode_64k", "op": "decode", "n": 1 << 16, "chunk": 512, "bits": 8, "mode": "quad", "data": "laplace"},
        # one 1024 x 1024 activation tensor
        {"name": "compress_1m", "op": "compress", "n": 1 << 20, "chunk": 2048, "bits": 8, "mode": "quad", "data": "gaussian"},
        {"name": "decode_1m", "op": "decode", "n": 1 << 20, "chunk": 2048, "bits": 8, "mode": "quad", "data": "gaussian"},
        # a shard of a gradient of average size, with a ragged end
        {"name": "compress_9m_ragged", "op": "compress", "n": 9 * (1 << 20) + 12325, "chunk": 2048, "bits": 8, "mode": "quad", "data": "student_t"},
        {"name": "decode_9m_ragged", "op": "decode", "n": 9 * (1 << 20) + 12325, "chunk": 2048, "bits": 8, "mode": "quad", "data": "student_t"},
        # a large request coded with the table of its tensor type
        {"name": "encode_48m_table", "op": "encode", "n": 48 * (1 << 20) + 32, "chunk": 1024, "bits": 8, "mode": "quad", "data": "gaussian"},
        # packed 6-bit (e3m2) weights read back
        {"name": "decode_e3m2_32m", "op": "decode", "n": 32 * (1 << 20) + 7, "chunk": 1024, "bits": 6, "mode": "m64a8", "data": "e3m2"},
        # the 8192 x 32768 activation tensor of the benchmark, both directions
        {"name": "compress_256m", "op": "compress", "n": 1 << 28, "chunk": 2048, "bits": 8, "mode": "quad", "data": "laplace"},
        {"name": "decode_256m", "op": "decode", "n": 1 << 28, "chunk": 2048, "bits": 8, "mode": "quad", "data": "laplace"},
        # the shards of one layer on one device's share of the batch, in one call each way
        {"name": "batch_encode_48", "op": "batch_encode", "tensors": 48, "lo": BATCH_LO, "hi": BATCH_HI, "sizes_seed": 2, "chunk": 2048, "bits": 8, "mode": "quad"},
        {"name": "batch_decode_48", "op": "batch_decode", "tensors": 48, "lo": BATCH_LO, "hi": BATCH_HI, "sizes_seed": 2, "chunk": 2048, "bits": 8, "mode": "quad"},
    ]


def draw(rng: random.Random):
    op = rng.choice(["compress", "compress", "encode", "decode", "decode", "table", "batch_encode", "batch_decode"])
    chunk = rng.choice([256, 512, 1024, 2048, 2048, 4096])
    if op.startswith("batch"):
        # 2^21 .. 2^28 symbols in all, in 2 .. 64 tensors whose sizes span a factor of 32
        tensors = int(round(2 ** rng.uniform(1, math.log2(BATCH_MAX_TENSORS))))
        hi = int(min(BATCH_HI, LARGEST // tensors, 2 ** rng.uniform(20, 25)))
        return {"op": op, "tensors": tensors, "lo": max(hi // 32, 1 << 15), "hi": hi, "sizes_seed": rng.randrange(1 << 16),
                "chunk": chunk, "bits": 8, "mode": "quad"}
    n = int(2 ** rng.uniform(math.log2(SMALLEST), math.log2(LARGEST)))
    if rng.random() < 0.5:
        n = n // 32 * 32                   # whole quantisation blocks; the others end anywhere
    bits = rng.choice([8, 8, 8, 8, 6, 4]) if op != "table" else 8
    if bits == 8:
        data = rng.choice(["gaussian", "laplace", "student_t", "weights", "uniform", "zeros90"])
        mode = rng.choice(["quad", "quad", "quad", "any", "paper_t1"])
    else:
        data, mode = ("e3m2", "m64a8") if bits == 6 else ("e2m1", "m16a4")
    return {"op": op, "n": n, "chunk": chunk, "bits": bits, "mode": mode, "data": data}


# ------------------------------------------------------------------ inputs
def _small_floats(n, bits, seed):
    """n packed codes of Laplace(0, 1) values in e2m1 (4 bits) or e3m2 (6 bits)."""
    exp_bits, mant_bits = (2, 1) if bits == 4 else (3, 2)
    mags = [(m / (1 << mant_bits)) if e == 0 else (1 + m / (1 << mant_bits)) * 2.0 ** (e - 1)
            for e in range(1 << exp_bits) for m in range(1 << mant_bits)]
    mid = torch.tensor([(a + b) / 2 for a, b in zip(mags, mags[1:])], dtype=torch.float32, device="cuda")
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    full = (n + 3) // 4 * 4
    e = torch.empty(full, device="cuda").exponential_(1.0, generator=g)
    sign = torch.randint(0, 2, (full,), generator=g, device="cuda", dtype=torch.int32)
    codes = torch.bucketize(e, mid, out_int32=True) + len(mags) * sign
    codes[n:] = 0
    if bits == 4:
        c = codes.view(-1, 2)
        packed = (c[:, 0] | (c[:, 1] << 4)).to(torch.uint8)
    else:
        c = codes.view(-1, 4)
        w = c[:, 0] | (c[:, 1] << 6) | (c[:, 2] << 12) | (c[:, 3] << 18)
        packed = torch.stack([w & 255, (w >> 8) & 255, (w >> 16) & 255], dim=1).to(torch.uint8).reshape(-1)
    return packed[:qlc.packed_bytes(n, bits)].contiguous()


def _tensor(n, data, bits, seed):
    """n symbols (packed for 4 and 6 bits) in a buffer of their own."""
    if bits != 8:
        return _small_floats(n, bits, seed)
    m = (n + 32767) // 32768 * 32768
    if data == "laplace":
        x = datagen.laplace_outlier_rows(m // 32768, 32768, seed, "cuda")
    elif data == "student_t":
        x = datagen.student_t(m, seed, "cuda")
    elif data == "weights":
        x = datagen.gaussian(m, seed, "cuda", std=0.02)
    elif data == "uniform":
        x = datagen.uniform_bytes(m, seed, "cuda")
    elif data == "zeros90":
        x = datagen.zeros90_gaussian(m, seed, "cuda")
    else:
        x = datagen.gaussian(m, seed, "cuda")
    return x[:n].clone()


def _batch_sizes(case):
    rng = random.Random(case["sizes_seed"])
    lo, hi = math.log(case["lo"]), math.log(case["hi"])
    return [int(max(32, 32 * round(math.exp(rng.uniform(lo, hi)) / 32))) for _ in range(case["tensors"])]


def _capacity(n, bits, mode):
    """Bitstream bytes: a searched table never needs more than the symbols themselves."""
    return qlc.qlc_encode_bound_bytes(n) if mode == "paper_t1" else (qlc.packed_bytes(n, bits) + 31) // 16 * 16


def _prepare_batch(case, seed):
    sizes = _batch_sizes(case)
    b = qlc.Batch(sizes, chunk_symbols=case["chunk"])
    for i, n in enumerate(sizes):
        b.input(i).copy_(datagen.shard(i, n, seed, "cuda"))
    ws = b.workspace()
    if case["op"] == "batch_decode":
        b.encode(ws, MODES[case["mode"]])
    return {"op": case["op"], "batch": b, "ws": ws, "mode": MODES[case["mode"]]}


def prepare(case, seed):
    if case["op"].startswith("batch"):
        return _prepare_batch(case, seed)
    n, bits, chunk, mode = case["n"], case["bits"], case["chunk"], MODES[case["mode"]]
    x = _tensor(n, case["data"], bits, seed)
    s = {"op": case["op"], "n": n, "bits": bits, "chunk": chunk, "mode": mode, "x": x,
         "table": qlc.new_table(), "ws": qlc.new_workspace(n, chunk)}
    if case["op"] == "table":
        return s
    s["stream"] = torch.zeros(_capacity(n, bits, case["mode"]), dtype=torch.uint8, device="cuda")
    s["index"] = torch.zeros(qlc.qlc_chunk_count(n, chunk), dtype=torch.int64, device="cuda")
    s["total"] = torch.zeros(1, dtype=torch.int64, device="cuda")
    s["err"] = torch.zeros(1, dtype=torch.int32, device="cuda")
    if case["op"] == "encode":
        # the type's table, from another tensor of it; codes may run longer than this tensor's own would
        k = min(n, 1 << 22)
        other = _tensor(k, case["data"], bits, seed + 7919)
        qlc.qlc_build_table_sym(other, k, bits, mode, s["table"], qlc.new_workspace(k, chunk))
        s["stream"] = torch.zeros(qlc.qlc_encode_bound_bytes(n), dtype=torch.uint8, device="cuda")
    elif case["op"] == "decode":
        _compress(s)
        s["out"] = torch.zeros_like(x)
        del s["x"]
    return s


# ------------------------------------------------------------------ one pass
def _compress(s):
    if s["bits"] == 8:
        qlc.qlc_compress(s["x"], s["mode"], s["table"], s["chunk"], s["stream"], s["index"], s["total"], s["err"], s["ws"])
    else:
        qlc.qlc_compress_sym(s["x"], s["n"], s["bits"], s["mode"], s["table"], s["chunk"], s["stream"], s["index"],
                             s["total"], s["err"], s["ws"])


def run(s):
    op = s["op"]
    if op == "compress":
        _compress(s)
        return [s["stream"], s["index"], s["total"], s["table"], s["err"]]
    if op == "encode":
        if s["bits"] == 8:
            qlc.qlc_encode(s["x"], s["table"], s["chunk"], s["stream"], s["index"], s["total"], s["err"], s["ws"])
        else:
            qlc.qlc_encode_sym(s["x"], s["n"], s["bits"], s["table"], s["chunk"], s["stream"], s["index"], s["total"],
                               s["err"], s["ws"])
        return [s["stream"], s["index"], s["total"], s["err"]]
    if op == "decode":
        if s["bits"] == 8:
            qlc.qlc_decode(s["stream"], s["total"], s["index"], s["chunk"], s["table"], s["n"], s["out"], s["err"], s["ws"])
        else:
            qlc.qlc_decode_sym(s["stream"], s["total"], s["index"], s["chunk"], s["table"], s["n"], s["bits"], s["out"],
                               s["err"], s["ws"])
        return [s["out"], s["err"]]
    if op == "table":
        qlc.qlc_build_table(s["x"], s["mode"], s["table"], s["ws"])
        return [s["table"]]
    b = s["batch"]
    if op == "batch_encode":
        b.encode(s["ws"], s["mode"])
        return [b.bits, b.index, b.total, b.tables, b.err]
    b.decode(s["ws"])
    return [b.out, b.err]


# ------------------------------------------------------------------ what a pass cannot do without
def work(case):
    if case["op"].startswith("batch"):
        sizes = _batch_sizes(case)
        n, count, bits, rate = sum(sizes), len(sizes), 8, 6.72
    else:
        n, count, bits, rate = case["n"], 1, case["bits"], CODE_BITS[case["data"]]
        if case["mode"] == "paper_t1" and case["data"] in ("uniform", "zeros90"):
            rate = 9.59 if case["data"] == "uniform" else 6.07
    plain, coded = n * bits / 8, n * rate / 8 + 8 * n / case["chunk"]
    if case["op"] == "table":
        coded = 0
    return {"bytes": float(plain + coded + count * qlc.TABLE_BYTES), "flops": 0.0}


def exact(case, seed):
    """Every output is bytes or whole numbers, which stay equal: there is nothing to round."""
    return None
