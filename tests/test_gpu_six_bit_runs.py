"""Decoded 6-bit symbols on both sides of the output size, and of the chunk
size, that choose how a wave's runs are stored: the decoded buffer is the
encoded one, byte for byte, and nothing is written behind it."""
import pytest
import torch

from paper_2602_17849_amd import qlc

pytestmark = pytest.mark.gpu

from gpu_util import DEV  # noqa: E402

EDGE = (40 << 20) * 8 // 6          # the most symbols whose packed bytes are 40 MiB


def _packed(n, seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    x = torch.randint(0, 256, (qlc.packed_bytes(n, 6),), generator=g, device=DEV,
                      dtype=torch.uint8)
    x[x.numel() // 3:x.numel() // 2] = 0            # short codes too
    if n * 6 % 8:
        x[-1] &= (1 << (n * 6 % 8)) - 1
    return x


@pytest.mark.parametrize("C", [256, 512])
@pytest.mark.parametrize("n", [EDGE, EDGE + 1])
def test_output_sizes(n, C):
    x = _packed(n, C)
    t, ws = qlc.new_table(), qlc.new_workspace(n, C)
    bits = torch.zeros(qlc.qlc_encode_bound_bytes(n), dtype=torch.uint8, device=DEV)
    index = torch.zeros(qlc.qlc_chunk_count(n, C), dtype=torch.int64, device=DEV)
    total = torch.zeros(1, dtype=torch.int64, device=DEV)
    err = torch.full((2,), -1, dtype=torch.int32, device=DEV)
    out = torch.full((x.numel() + 64,), 0xAA, dtype=torch.uint8, device=DEV)
    qlc.qlc_compress_sym(x, n, 6, qlc.LAYOUT_M64_AREAS8, t, C, bits, index, total, err[:1], ws)
    qlc.qlc_decode_ex(bits, total, index, C, t, n, 6, qlc.DECODER_LANE, out, err[1:], ws)
    torch.cuda.synchronize()
    assert err.tolist() == [0, 0]
    assert torch.equal(out[:x.numel()], x)
    assert (out[x.numel():] == 0xAA).all()


@pytest.mark.parametrize("C", [256, 512])
def test_batched(C):
    sizes = [1 << 20, 70001, 64 * C, 64 * C + 8, 5]
    b = qlc.Batch(sizes, chunk_symbols=C)
    b.out.fill_(0xAA)
    xs = [_packed(n, i) for i, n in enumerate(sizes)]
    for i, x in enumerate(xs):
        b.input(i)[:x.numel()] = x
    tun = qlc.BatchTuning(0, 0, 0, qlc.DECODER_LANE)
    ws = b.workspace(tun)
    qlc.qlc_encode_batched_sym(b.jobs, b.S, 6, qlc.LAYOUT_M64_AREAS8, C, ws, tun)
    qlc.qlc_decode_batched_sym(b.jobs, b.S, 6, C, ws, tun)
    torch.cuda.synchronize()
    assert b.err.tolist() == [0] * b.S
    for i, x in enumerate(xs):
        o = b.output(i)
        assert torch.equal(o[:x.numel()], x), i
        assert (o[x.numel():] == 0xAA).all(), i
