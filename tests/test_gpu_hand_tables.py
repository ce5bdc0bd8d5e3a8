"""Decodes with tables that no call of the library builds: made by hand, as a
program may write any table record into device memory.  Tolerance zero."""
import numpy as np
import pytest
import torch

import oracle
from paper_2602_17849_amd import datagen, qlc

pytestmark = pytest.mark.gpu

from gpu_util import gpu_decode, table_from_oracle, to_dev  # noqa: E402

R2S = 512       # byte offset of rank_to_sym in a table


@pytest.mark.parametrize("decoder", [qlc.DECODER_LANE, qlc.DECODER_SPLIT])
@pytest.mark.parametrize("rem", [0, 5])
@pytest.mark.parametrize("bits,A,p", [(4, 4, 2), (6, 8, 3)])
def test_symbols_outside_the_alphabet(bits, A, p, rem, decoder):
    """Ranks that name symbols above the alphabet's: the decoded field is the
    symbol's low bits, and the symbols beside it are as they would be."""
    M, C = 1 << bits, 256
    n = C * 70 + 64 + rem
    x = np.random.default_rng(bits).integers(0, M, n, dtype=np.uint8)
    ot = oracle.build_table_general(np.arange(M, 0, -1, dtype=np.uint64), M, A, p, A)
    st, stream, index, total = oracle.encode(x, ot, C)
    assert st == 0
    tab = table_from_oracle(ot).cpu().numpy().copy()
    tab[R2S:R2S + M:3] |= 0xFF & ~(M - 1)
    tab[R2S + 1:R2S + M:3] |= M
    err, out = gpu_decode(stream, total, index, C, to_dev(tab), n, decoder, bits)
    assert err == 0
    assert np.array_equal(out, datagen.pack_symbols(x, bits))
