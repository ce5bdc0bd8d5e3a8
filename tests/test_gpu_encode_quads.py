"""The encoder where its packing and its loading can go wrong: groups of four
codes from 4 to 44 bits (two words or three), codes of one to eleven bits
before a segment's first word, and inputs that end at and around the edges of
its runs of 16, half tiles of 4096, tiles and segments of 8192 symbols,
against the oracle.  Tolerance zero."""
import numpy as np
import pytest
import torch

import oracle
from paper_2602_17849_amd import datagen, qlc

pytestmark = pytest.mark.gpu

from gpu_util import DEV, gpu_encode, table_from_oracle, to_dev  # noqa: E402

# past a segment of 8192 symbols: nothing, part of a run, runs, half a tile
ENDS = [1, 8191, 8192, 8193, 8207, 8208, 8209, 12287, 12288, 12289, 12303, 16383, 24576 + 4111]


@pytest.mark.parametrize("p_long", [0.0, 0.1, 1.0])
@pytest.mark.parametrize("n", ENDS)
def test_code_lengths_bytes(n, p_long):
    """One symbol of 3 bits, the others 11: quads of 12, 20 .. 44 bits."""
    hist = np.ones(256, dtype=np.uint64)
    hist[0] = 1 << 40
    ot = oracle.build_table(hist, qlc.LAYOUT_SEARCH_QUAD)
    rng = np.random.default_rng(n)
    x = np.where(rng.random(n) < p_long, rng.integers(1, 256, n), 0).astype(np.uint8)
    st, obits, oindex, ototal = oracle.encode(x, ot, 512)
    assert st == 0
    err, bits, nbytes, index, total = gpu_encode(to_dev(x), table_from_oracle(ot), 512)
    assert err == 0 and total == ototal
    assert np.array_equal(bits[:nbytes], obits) and not bits[nbytes:].any()
    assert np.array_equal(index, oindex)


@pytest.mark.parametrize("bits,mode,M,A,p", [(4, qlc.LAYOUT_M16_AREAS2, 16, 2, 1),
                                             (6, qlc.LAYOUT_M64_AREAS8, 64, 8, 3)])
@pytest.mark.parametrize("n", ENDS)
def test_compress_small_alphabets(n, bits, mode, M, A, p):
    """Packed input; with 2 areas a code is 1 bit or more, so 32 symbols
    before a segment are what its first word needs."""
    C = 256
    rng = np.random.default_rng(n + bits)
    x = np.where(rng.random(n) < 0.05, rng.integers(0, M, n), 0).astype(np.uint8)
    xd = to_dev(datagen.pack_symbols(x, bits))
    ot = oracle.build_table_general(np.bincount(x, minlength=M).astype(np.uint64), M, A, p, 8)
    st, obits, oindex, ototal = oracle.encode(x, ot, C)
    assert st == 0
    cap = qlc.qlc_encode_bound_bytes(n)
    stream = torch.zeros(cap, dtype=torch.uint8, device=DEV)
    index = torch.zeros(qlc.qlc_chunk_count(n, C), dtype=torch.int64, device=DEV)
    total = torch.zeros(1, dtype=torch.int64, device=DEV)
    err = torch.full((1,), -1, dtype=torch.int32, device=DEV)
    qlc.qlc_compress_sym(xd, n, bits, mode, qlc.new_table(), C, stream, index, total, err,
                         qlc.new_workspace(n, C))
    torch.cuda.synchronize()
    assert int(err.item()) == 0 and int(total.item()) == ototal
    got = stream.cpu().numpy()
    assert np.array_equal(got[:obits.size], obits) and not got[obits.size:].any()
    assert np.array_equal(index.cpu().numpy().astype(np.uint64), oindex)
