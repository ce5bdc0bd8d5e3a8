"""The lane decoder's position arithmetic on the host (its header, compiled
with the host compiler): the refill schedule of a chunk walked over valid
index entries and over wrong ones, among them entries 2^32 bits and more from
the wave's base.  A wrong entry has to end like any other, and wherever a
lane starts, every bit that a window reads before the chunk's end has to be
in its ring."""
import ctypes
import os
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2602_17849_amd", "csrc")

WALK = r"""
#define __host__
#define __device__
#define __forceinline__ inline
#include "qlc_lane_pos.h"
using namespace qlc;

struct Wave {                   // one lane; what a slot of the ring holds
  LanePos& L;
  uint64_t rel0;
  uint64_t* slot;               // absolute first bit of its superblock
  uint64_t* flight;             // requested, not arrived (~0: nothing)
  uint32_t* polls;              // turns of the loop for one refill
  uint32_t* group;              // groups decoded, now and at the last request
  bool* waited;                 // for a superblock asked for less than four groups ago
  bool any(bool b) const { return b && ++*polls < 100; }
  void arrive() const {
    if (*flight != ~0ull) {
      slot[(*flight >> kSbLog2Bits) & 3] = *flight;
      *waited |= group[0] < group[1] + 4;
    }
    *flight = ~0ull;
    L.arrived();
  }
  void request() const {
    const bool need = L.wants();
    if (need) *flight = rel0 + 8ull * L.load_offset();
    group[1] = group[0];
    L.requested(need);
  }
};

// Codes of len[k % nlen] bits from pos0 on.  0: every window was served;
// 1: a refill that does not end; 2: a bit missing from the ring; 3: a load
// offset past the limit; 4: the position is not the sum of the lengths; 5: a
// wait for a superblock that was asked for less than four groups ago.
extern "C" int walk(uint64_t rel0, uint64_t pos0, uint64_t end, uint32_t groups,
                    const uint8_t* len, uint32_t nlen) {
  LanePos L;
  uint64_t slot[4] = {~0ull, ~0ull, ~0ull, ~0ull}, flight = ~0ull;
  uint32_t polls = 0, group[2] = {0, 0};
  bool waited = false;
  L.start(true, rel0, pos0, end);
  for (int s = 0; s < 2; ++s) {
    const uint64_t a = rel0 + 8ull * L.load_offset();
    slot[(a >> kSbLog2Bits) & 3] = a;
    L.requested(true);
  }
  L.arrived();
  const Wave w{L, rel0, slot, &flight, &polls, group, &waited};
  w.request();
  uint64_t pos = pos0;
  uint32_t k = 0;
  for (uint32_t g = 0; g < groups; ++g) {
    // the group's window: 96 bits from pos on
    for (uint64_t sb = pos & ~(uint64_t)(kSbBits - 1); sb < pos + 96 && sb < end; sb += kSbBits)
      if (slot[(sb >> kSbLog2Bits) & 3] != sb) return 2;
    uint32_t adv = 0;
    for (int i = 0; i < 8; ++i) adv += len[k++ % nlen];
    L.q += adv;
    pos += adv;
    if (L.base(rel0) + L.q + 1 != pos) return 4;
    polls = 0;
    group[0] = g + 1;
    if ((g & 7) == 3) lane_mid(L, w);
    if ((g & 7) == 7) lane_refill(L, w);
    if (waited) return 5;
    if (polls >= 100) return 1;
    if (L.load_offset() >= kOobOffset) return 3;
  }
  return 0;
}
extern "C" uint64_t max_lane_sb() { return kMaxLaneSb; }
extern "C" bool balance(uint64_t blocks, uint32_t cus) { return lane_balance(blocks, cus); }
"""


@pytest.fixture(scope="module")
def walk(tmp_path_factory):
    d = tmp_path_factory.mktemp("lane_pos")
    (d / "walk.cpp").write_text(WALK)
    so = str(d / "walk.so")
    subprocess.check_call(["g++", "-O1", "-std=c++17", "-Wall", "-fPIC", "-shared", "-I" + CSRC,
                           str(d / "walk.cpp"), "-o", so])
    lib = ctypes.CDLL(so)
    u64, u32 = ctypes.c_uint64, ctypes.c_uint32
    lib.walk.argtypes = [u64, u64, u64, u32, ctypes.c_char_p, u32]
    lib.max_lane_sb.restype = u64

    def run(rel0, pos0, end, groups, lens):
        b = bytes(int(v) for v in lens)
        return lib.walk(rel0, pos0, end, groups, b, len(b))
    run.max_sb = lib.max_lane_sb()
    lib.balance.argtypes, lib.balance.restype = [u64, u32], ctypes.c_bool
    run.balance = lib.balance
    return run


def _lens(kind, rng):
    return {"11": [11], "1": [1], "8": [8], "runs": [11] * 777 + [1] * 500 + [6] * 100,
            "any": rng.integers(1, 12, 4096)}[kind]


@pytest.mark.parametrize("kind", ["11", "1", "8", "runs", "any"])
@pytest.mark.parametrize("C", [256, 2048, 65536])
def test_valid_chunks(walk, kind, C):
    rng = np.random.default_rng(C)
    lens = _lens(kind, rng)
    total = int(sum(int(lens[k % len(lens)]) for k in range(C)))
    for _ in range(40):
        rel0 = 2048 * int(rng.integers(0, 1 << 40))
        pos0 = rel0 + int(rng.integers(0, 64 * 65536 * 11))
        assert walk(rel0, pos0, pos0 + total, C // 8, lens) == 0


# distances of a lane's first bit from the wave's base at which 32-bit sums
# wrap, and the last ones that a wave accepts
FAR = [2**31, 2**32 - 2048, 2**32 - 1537, 2**32 - 1024, 2**32 - 512, 2**32 - 392, 2**32 - 88,
       2**32 - 1, 2**32, 2**32 + 777, 3 * 2**32 - 1200]


@pytest.mark.parametrize("far", FAR + ["last"])
@pytest.mark.parametrize("kind", ["11", "1", "any"])
def test_entries_far_from_the_base(walk, far, kind):
    """The wave's first entry too low: its other chunks are whole, and decode
    as they would from any base."""
    rng = np.random.default_rng(3)
    lens = _lens(kind, rng)
    C = 65536
    total = int(sum(int(lens[k % len(lens)]) for k in range(C)))
    for d in [0, 1, 2, 3, 5, 88, 700, 40000]:
        pos0 = (walk.max_sb << 9) - d if far == "last" else far - d
        for rel0 in (0, 2048 * 12345):
            assert walk(rel0, rel0 + pos0, rel0 + pos0 + total, C // 8, lens) == 0


def test_wrong_ends(walk):
    """Ends before, at and long after where the codes end."""
    rng = np.random.default_rng(5)
    for _ in range(4000):
        rel0 = 2048 * int(rng.integers(0, 1 << 30))
        pos0 = rel0 + int(rng.choice(FAR)) - int(rng.integers(0, 4096))
        end = pos0 + int(rng.choice([0, 1, 511, 512, 4096, 2**31, 2**32 - 1, 2**32, 2**34])) \
            + int(rng.integers(0, 3000))
        assert walk(rel0, pos0, end, 64, _lens(str(rng.choice(["11", "1", "any"])), rng)) == 0


def test_random_entries(walk):
    rng = np.random.default_rng(6)
    lens = _lens("any", rng)
    for _ in range(20000):
        pos0 = int(rng.integers(0, 1 << 35)) % (walk.max_sb << 9)
        end = pos0 + int(rng.integers(0, 1 << 36))
        assert walk(0, pos0, end, 32, lens) == 0


@pytest.mark.parametrize("cus", [32, 64, 256, 304])
def test_balanced_launches(walk, cus):
    """Only launches that fit the device at once, whatever its size."""
    assert not walk.balance(1, cus) and not walk.balance(cus, cus)
    assert walk.balance(cus + 1, cus) and walk.balance(2 * cus, cus)
    assert not walk.balance(2 * cus + 1, cus) and not walk.balance(1 << 33, cus)
