"""CPU model of the split decoder's boundary search with the corrections that
its kernel makes: a lane whose start is not where the lane before it left
walks its whole piece again from there, with 32 or with 64 codes per lane.
On streams the oracle writes: the rounds end within G + 1, every piece starts
at a code, and the counts sum to the chunk's symbols."""
import math

import numpy as np
import pytest

import oracle

WARM = 512          # bits walked before a piece, not counted


def _lengths(t, sb):
    """Code length of the code starting at every bit of the stream sb."""
    p = t.prefix_bits
    w = np.array([min(int(v), 8) for v in t.width])
    area = np.zeros(sb.size - 3, dtype=np.int64)
    for i in range(p):
        area = (area << 1) | sb[i:i + area.size]
    return (p + w[area]).tolist()


def _walk(lens, x, stop):
    c = 0
    while x < stop:
        x += lens[x]
        c += 1
    return x, c


def boundaries(lens, s, e, G, d):
    """Start and code count of each of a chunk's G pieces, and the rounds."""
    n = e - s
    piece = (n + G - 1) // G
    start, end, exits, cnt = [], [], [], []
    for g in range(G):
        a, b = min(g * piece, n), min((g + 1) * piece, n)
        u = (max(a - WARM, 0) + d - 1) // d * d
        st, _ = _walk(lens, s + u, s + a)
        x, c = _walk(lens, st, s + b)
        start.append(st), end.append(s + b), exits.append(x), cnt.append(c)
    rounds = 0
    while True:
        prev, changed = [s] + exits[:-1], False
        for g in range(1, G):
            if prev[g] != start[g]:
                x, cnt[g] = _walk(lens, prev[g], end[g])
                changed |= x != exits[g]
                exits[g], start[g] = x, prev[g]
        rounds += 1
        assert rounds <= G + 1
        if not changed:
            return start, cnt, exits[-1], rounds


def _check(x, t, C, per_lane):
    st, bits, index, total = oracle.encode(x, t, C)
    assert st == 0
    sb = np.concatenate([np.unpackbits(np.asarray(bits, np.uint8)), np.zeros(512, np.uint8)])
    lens = _lengths(t, sb)
    d = math.gcd(*(t.prefix_bits + min(int(w), 8) for w, c in zip(t.width, t.count) if c))
    at = np.concatenate([[0], np.cumsum(np.asarray(t.len)[x])])     # true code starts
    most = 0
    for j, s in enumerate(index):
        e = int(index[j + 1]) if j + 1 < len(index) else total
        first, nsym = j * C, min(C, x.size - j * C)
        start, cnt, last, rounds = boundaries(lens, int(s), e, C // per_lane, d)
        assert sum(cnt) == nsym and last == e
        k = first
        for s0, c in zip(start, cnt):
            assert c == 0 or s0 == at[k]
            k += c
        most = max(most, rounds)
    return most


@pytest.mark.parametrize("per_lane,C", [(32, 256), (32, 2048), (32, 8192), (64, 256), (64, 2048),
                                        (64, 16384)])
def test_rounds_and_starts(per_lane, C):
    rng = np.random.default_rng(C + per_lane)
    n = 2 * max(C, 4096) + 77
    x = np.clip(np.round(rng.laplace(128, 6, n)), 0, 255).astype(np.uint8)
    for mode in (0, 2, 3):
        _check(x, oracle.build_table(oracle.histogram(x), mode), C, per_lane)
    u = rng.integers(0, 256, n).astype(np.uint8)                    # one code length
    assert _check(u, oracle.build_table(oracle.histogram(u), 0), C, per_lane) == 1
    z = np.where(rng.random(n) < 0.003, x, 128).astype(np.uint8)    # nearly all one value
    _check(z, oracle.build_table(oracle.histogram(z), 0), C, per_lane)


@pytest.mark.parametrize("per_lane", [32, 64])
def test_never_in_step(per_lane):
    """Nearly one symbol, under a table of several lengths: a wrong start never
    falls in step, and each round makes one more lane exact."""
    C = 2048
    x = np.zeros(2 * C, np.uint8)
    x[:40] = np.arange(40)
    G = C // per_lane
    t = oracle.build_table(oracle.histogram(x), 0)
    assert G // 2 <= _check(x, t, C, per_lane) <= G + 1


@pytest.mark.parametrize("M,A,p", [(16, 2, 1), (16, 4, 2), (64, 8, 3)])
def test_small_alphabets(M, A, p):
    x = np.minimum(np.random.default_rng(3).geometric(0.3, 7001) - 1, M - 1).astype(np.uint8)
    t = oracle.build_table_general(oracle.histogram(x)[:M], M, A, p, A)
    for per_lane in (32, 64):
        _check(x, t, 512, per_lane)
