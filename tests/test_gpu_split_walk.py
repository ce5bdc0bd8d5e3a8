"""The split decoder's length walk and the decoders' LUT build where they can
go wrong: code lengths from 1 to 11 bits (what fills the walk's 64-bit
register), both counts of codes per lane on either side of the tensor size
that chooses between them, and tables whose areas are not back to back,
against the oracle or against a plain decode of the table's documented
meaning.  Tolerance zero."""
import numpy as np
import pytest
import torch

import oracle
from paper_2602_17849_amd import datagen, qlc

pytestmark = pytest.mark.gpu

from gpu_util import DEV, gpu_decode, gpu_encode, gpu_table, table_from_oracle, to_dev  # noqa: E402


@pytest.mark.parametrize("C", [256, 8192, 16384])
@pytest.mark.parametrize("n", [(2 << 20) - 5, 2 << 20, (2 << 20) + 5])
def test_codes_per_lane(n, C):
    """32 codes per lane up to 2 Mi symbols (C <= 8192), 64 beyond."""
    x = datagen.gaussian((n + 31) // 32 * 32, seed=C)[:n].numpy()
    xd = to_dev(x)
    t = gpu_table(xd, qlc.LAYOUT_SEARCH_QUAD)
    err, bits, nbytes, index, total = gpu_encode(xd, t, C)
    assert err == 0
    err, out = gpu_decode(bits[:nbytes], total, index, C, t, n, qlc.DECODER_SPLIT)
    assert err == 0
    assert np.array_equal(out, x)


@pytest.mark.parametrize("p_long", [0.0, 0.02, 0.5, 1.0])
@pytest.mark.parametrize("widths", ["steep", "t2", "m16"])
def test_walk_code_lengths(widths, p_long):
    """steep: one symbol of 3 bits, the others 11; t2: 4, 6, 8 and 11 bits;
    m16: 1 and 5 bits (16 symbols in 2 areas)."""
    C, n = 1024, 1024 * 21 + 77
    rng = np.random.default_rng(int(100 * p_long))
    m16 = widths == "m16"
    M = 16 if m16 else 256
    hist = np.ones(M, dtype=np.uint64)
    hist[0] = 1 << 40
    if widths == "t2":
        ot = oracle.build_table(hist, qlc.LAYOUT_PAPER_T2)
    elif m16:
        ot = oracle.build_table_general(hist, M, 2, 1, 8)
    else:
        ot = oracle.build_table(hist, qlc.LAYOUT_SEARCH_QUAD)
    lens = np.asarray(ot.len)[:M]
    rare = np.flatnonzero(lens == lens.max())
    x = np.where(rng.random(n) < p_long, rng.choice(rare, n), 0).astype(np.uint8)
    st, bits, index, total = oracle.encode(x, ot, C)
    assert st == 0
    bits_per = 4 if m16 else 8
    for dec in (qlc.DECODER_SPLIT, qlc.DECODER_LANE):
        err, out = gpu_decode(bits, total, index, C, table_from_oracle(ot), n, dec, bits_per)
        assert err == 0, dec
        assert np.array_equal(out, datagen.pack_symbols(x, bits_per)), dec


def _plain_decode(t, stream_bits, C, n):
    """Decode n codes of a bit array by the table's meaning: the area code,
    its suffix, and the last area whose code range holds the word and whose
    rank it holds.  Returns symbols, index, total bits, any invalid code."""
    w = [min(int(v), 8) for v in t["width"]]
    out, index, pos, bad = [], [], 0, False
    for i in range(n):
        if i % C == 0:
            index.append(pos)
        a = int("".join(map(str, stream_bits[pos:pos + 3])), 2)
        ln = 3 + w[a]
        word = int("".join(map(str, stream_bits[pos:pos + ln])), 2)
        sym = None
        for k in range(8):
            lo = k << w[k]
            if lo <= word < lo + (1 << w[k]):
                r = int(t["offset"][k]) + word - lo
                if int(t["first"][k]) <= r < int(t["first"][k]) + int(t["count"][k]) and r < 256:
                    sym = int(t["rank_to_sym"][r])
        bad |= sym is None
        out.append(0 if sym is None else sym)
        pos += ln
    return np.array(out, np.uint8), np.array(index, np.int64), pos, bad


@pytest.mark.parametrize("kind", ["gap", "decreasing", "sum_over_256"])
@pytest.mark.parametrize("decoder", [1, 2])
def test_tables_not_back_to_back(kind, decoder):
    ot = oracle.build_table(np.arange(256, 0, -1, dtype=np.uint64), qlc.LAYOUT_PAPER_T1)
    raw = table_from_oracle(ot).cpu().numpy()
    tab = np.frombuffer(raw.tobytes(), dtype=np.uint8).copy()
    first = tab[1040:1056].view(np.uint16)
    count = tab[1056:1072].view(np.uint16)
    width, offset = tab[1024:1032], tab[1032:1040]
    if kind == "gap":              # area 2's ranks moved up: a hole before them
        first[2] += 3
        offset[2] += 3
    elif kind == "decreasing":     # area 1 wider than area 2
        width[1], count[1] = 4, 16
    else:                          # more ranks than symbols
        count[7] = 200
        first[7] = 88
    t = qlc.parse_table(tab.tobytes())
    C, n = 256, 256 * 5 + 9
    rng = np.random.default_rng(7)
    bits = rng.integers(0, 2, 16 * n).tolist()
    sym, index, total, bad = _plain_decode(t, bits, C, n)
    words = (total + 31) // 32
    stream = np.packbits(np.array(bits[:total] + [0] * (32 * words - total), np.uint8))
    err, out = gpu_decode(stream, total, index, C, to_dev(tab), n, decoder)
    assert err == (qlc.QLC_ERR_CORRUPT_STREAM if bad else 0)
    if not bad:
        assert np.array_equal(out, sym)
