"""An index whose wave's first entry is far too low, so that the wave's other,
whole chunks lie 2^32 bits and more behind it: the lane decoder reports the
corrupt stream, decodes the other chunks from their own entries, and ends."""
import numpy as np
import pytest
import torch

import oracle
from paper_2602_17849_amd import qlc

pytestmark = pytest.mark.gpu

from gpu_util import DEV, table_from_oracle, to_dev  # noqa: E402


@pytest.mark.parametrize("batched", [False, True])
@pytest.mark.parametrize("far", [0, 1, 2])
def test_first_entry_too_low(far, batched):
    C = 256
    n = 64 * C + 5 * C + 19
    x = np.random.default_rng(far).integers(88 if far else 0, 256, n, dtype=np.uint8)
    ot = oracle.build_table(np.arange(256, 0, -1, dtype=np.uint64), qlc.LAYOUT_PAPER_T1)
    st, bits, index, total = oracle.encode(x, ot, C)
    assert st == 0
    # the stream behind `shift` bits of zeros; half of its first wave's
    # chunks lie past a multiple of 2^32
    shift = ((far << 32) - total // 2) // 128 * 128 if far else 0
    buf = torch.zeros(shift // 8 + len(bits) + 64, dtype=torch.uint8, device=DEV)
    buf[shift // 8:shift // 8 + len(bits)] = to_dev(bits)
    idx = index.astype(np.int64) + shift
    idx[0] = 0
    idx, t = to_dev(idx), table_from_oracle(ot)
    tot = torch.tensor([total + shift], dtype=torch.int64, device=DEV)
    if batched:
        b = qlc.Batch([n], chunk_symbols=C)
        j = b.jobs_host[0]
        j.table, j.bits, j.chunk_index = t.data_ptr(), buf.data_ptr(), idx.data_ptr()
        j.total_bits, j.bits_capacity, j.build_table = tot.data_ptr(), buf.numel(), 0
        b.upload_jobs()
        tun = qlc.BatchTuning(0, 0, 0, qlc.DECODER_LANE)
        b.decode(b.workspace(tun), tun)
        torch.cuda.synchronize()
        err, out = int(b.err[0].item()), b.output(0).cpu().numpy()
    else:
        out = torch.full((n,), 0xAA, dtype=torch.uint8, device=DEV)
        e = torch.full((1,), -1, dtype=torch.int32, device=DEV)
        qlc.qlc_decode_ex(buf, tot, idx, C, t, n, 8, qlc.DECODER_LANE, out, e,
                          qlc.new_workspace(0, C))
        torch.cuda.synchronize()
        err, out = int(e.item()), out.cpu().numpy()
    assert err == (qlc.QLC_ERR_CORRUPT_STREAM if far else 0)
    assert np.array_equal(out[C if far else 0:], x[C if far else 0:])
