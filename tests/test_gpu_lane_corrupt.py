"""One flipped bit in a stream with a sound index, at a place where the result
is determined: the first bit of a code, whose area code then names a code of
another length, in a chunk whose end a walk over the flipped bits misses.  The
lane decoder reports it, and every other chunk decodes as before,
on both sides of the workgroup counts at which a launch evens out its waves."""
import numpy as np
import pytest
import torch

import oracle
from paper_2602_17849_amd import qlc

pytestmark = pytest.mark.gpu

from gpu_util import gpu_decode, gpu_encode, table_from_oracle, to_dev  # noqa: E402

C = 256


def _end(bits, pos, width, nsym):
    """Where nsym codes from bit pos on end."""
    for _ in range(nsym):
        a = 0
        for k in range(3):
            a = 2 * a + (int(bits[(pos + k) >> 3]) >> (7 - ((pos + k) & 7)) & 1)
        pos += 3 + int(width[a])
    return pos


@pytest.mark.parametrize("blocks", [1, 256, 257, 512, 513])
@pytest.mark.parametrize("where", ["first", "middle", "short"])
def test_flipped_area_code(blocks, where):
    n = (blocks - 1) * 256 * C + 100 * C + 203
    rng = np.random.default_rng(blocks)
    x = np.where(np.arange(n) // 100 % 2 == 1, rng.integers(88, 256, n, dtype=np.uint8),
                 rng.integers(0, 40, n, dtype=np.uint8))
    ot = oracle.build_table(np.arange(256, 0, -1, dtype=np.uint64), qlc.LAYOUT_PAPER_T1)
    t = table_from_oracle(ot)
    err, bits, nbytes, index, total = gpu_encode(to_dev(x), t, C)
    assert err == 0
    bits = bits[:nbytes]
    j = {"first": 0, "middle": len(index) // 2, "short": len(index) - 1}[where]
    end = int(index[j + 1]) if j + 1 < len(index) else total
    nsym = min(C, n - j * C)
    assert _end(bits, int(index[j]), ot.width, nsym) == end
    for k in range(nsym):
        at = _end(bits, int(index[j]), ot.width, k)
        bad = bits.copy()
        bad[at >> 3] ^= 0x80 >> (at & 7)
        if _end(bad, at, ot.width, nsym - k) != end:
            break
    else:
        pytest.fail("no such code in the chunk")
    err, out = gpu_decode(bad, total, index, C, t, n, qlc.DECODER_LANE)
    assert err == qlc.QLC_ERR_CORRUPT_STREAM
    same = np.ones(n, bool)
    same[j * C:j * C + nsym] = False
    assert np.array_equal(out[same], x[same])
