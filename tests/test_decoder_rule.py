"""The line between the two decoders that QLC_DECODER_AUTO draws: near it the
split decoder may not be chosen, because tensors that are nearly all one value
take it several times as long as one lane per chunk."""
import pytest

from paper_2602_17849_amd import qlc

# the least n at each C for which the lane decoder is taken
LINE = {256: 2182187, 512: 9789474, 1024: 25004049, 2048: 55434009, 4096: 116293928,
        8192: 238012956, 16384: 481451013}


@pytest.mark.parametrize("C", sorted(LINE))
def test_line(C):
    ch = qlc.qlc_decoder_choice
    assert ch(LINE[C] - 1, C) == qlc.DECODER_SPLIT
    assert ch(LINE[C], C) == qlc.DECODER_LANE
    for n in (0, 1, 1 << 16, LINE[C] // 2):
        assert ch(n, C) == qlc.DECODER_SPLIT
    for k in (1.05, 1.15, 1.5, 8):
        assert ch(int(LINE[C] * k), C) == qlc.DECODER_LANE


@pytest.mark.parametrize("C", [32768, 65536])
def test_long_chunks(C):
    for n in (0, 1 << 16, 1 << 30):
        assert qlc.qlc_decoder_choice(n, C) == qlc.DECODER_LANE
