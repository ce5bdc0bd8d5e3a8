"""The lane decoder's refill: what its ring holds when codes run longer or
shorter than the one superblock per eight groups that it normally takes, and
launches on both sides of the workgroup counts at which it evens out the
waves of a SIMD.  Streams from the oracle (tolerance zero), or from the
encoder where the tensor is too large for it (the encoder's own parity is
tested elsewhere): the decoded bytes are the input."""
import numpy as np
import pytest
import torch

import oracle
from paper_2602_17849_amd import qlc

pytestmark = pytest.mark.gpu

from gpu_util import DEV, gpu_decode, gpu_encode, table_from_oracle, to_dev  # noqa: E402


def _table():
    """Table 1's widths (codes of 6, 7, 8 and 11 bits), ranks = symbols."""
    hist = np.arange(256, 0, -1, dtype=np.uint64)
    return oracle.build_table(hist, qlc.LAYOUT_PAPER_T1)


def _symbols(kind, n, seed):
    """Symbol = rank: ranks 0..39 take 6 bits, 88..255 take 11."""
    rng = np.random.default_rng(seed)
    short = rng.integers(0, 40, n, dtype=np.uint8)
    long_ = rng.integers(88, 256, n, dtype=np.uint8)
    if kind == "long":
        return long_
    if kind == "short":
        return short
    run = int(kind.split("_")[1])                # runs of one length, phase by seed
    pick = ((np.arange(n) + 37 * seed) // run) & 1
    return np.where(pick == 1, long_, short)


@pytest.mark.parametrize("C", [256, 2048])
@pytest.mark.parametrize("kind", ["long", "short", "runs_32", "runs_64", "runs_100", "runs_777"])
def test_lane_rates(kind, C):
    n = C * 64 + 5 * C + 19                      # a whole wave and a partial one
    x = _symbols(kind, n, seed=len(kind))
    ot = _table()
    st, bits, index, total = oracle.encode(x, ot, C)
    assert st == 0
    err, out = gpu_decode(bits, total, index, C, table_from_oracle(ot), n, qlc.DECODER_LANE)
    assert err == 0
    assert np.array_equal(out, x)


@pytest.mark.parametrize("blocks", [256, 257, 512, 513])
def test_lane_workgroup_counts(blocks):
    """blocks workgroups of 256 chunks, the last one short, mixed code lengths."""
    C = 256
    n = (blocks - 1) * 256 * C + 100 * C + 3
    x = _symbols("runs_100", n, seed=blocks)
    xd = to_dev(x)
    t = table_from_oracle(_table())
    err, bits, nbytes, index, total = gpu_encode(xd, t, C)
    assert err == 0
    err, out = gpu_decode(bits[:nbytes], total, index, C, t, n, qlc.DECODER_LANE)
    assert err == 0
    assert np.array_equal(out, x)
    bits[nbytes // 2] ^= 0x10                    # a corrupt stream ends all the same
    err, _ = gpu_decode(bits[:nbytes], total, index, C, t, n, qlc.DECODER_LANE)
    assert err in (0, qlc.QLC_ERR_CORRUPT_STREAM)
