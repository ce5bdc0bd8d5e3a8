// Positions of a lane of the one-lane-per-chunk decoder: where it is in its
// chunk's bits, what its ring holds and what it has requested.  Plain
// arithmetic, apart from the kernel, so that a program on the host can walk
// it over any index entry, valid or not.
#pragma once

#include <stdint.h>

namespace qlc {

constexpr uint32_t kSbLog2Bits = 9;        // superblock: 512 bits = 64 bytes
constexpr uint32_t kSbBits = 1u << kSbLog2Bits;
constexpr uint32_t kRingBits = 4 * kSbBits;  // ring of four superblocks
constexpr uint32_t kLookaheadBits = 3 * kSbBits;  // request a superblock up to three ahead
constexpr uint32_t kReach = 3 * 88 + 128;  // bits past q that four groups' windows may read
constexpr uint32_t kDue = 4 * 88 + kReach;  // ... and that they may read four groups later
static_assert(kReach + kSbBits <= kLookaheadBits, "a lane can always request what it may need");
constexpr uint32_t kOobOffset = 0xFFFFF000u;  // load offset of no request (room for what is added)
// A lane's first bit lies at most this many superblocks after its wave's
// base: the byte offsets of its loads stay below kOobOffset.
constexpr uint64_t kMaxLaneSb = (kOobOffset >> (kSbLog2Bits - 3)) - 4096;

// All positions are relative to the lane's own base, a multiple of the ring
// at or before its first bit (so that they are also the ring's).  A chunk is
// at most 65536 codes of 11 bits and the end is capped, so that no sum of
// them wraps whatever the index holds: relative to the wave's base they did,
// for an entry 2^32 bits away, and a lane whose request had wrapped waited
// for bits that it never asked for.
constexpr uint32_t kMaxEnd = 1u << 30;

struct LanePos {
  uint32_t q;        // bit of the next symbol, minus one
  uint32_t F;        // first bit not requested yet (a multiple of kSbBits)
  uint32_t have;     // first bit that is not in the ring yet
  uint32_t endr;     // end of the chunk: nothing is requested from there on
  uint32_t off;      // byte of the lane's base after the wave's base

  // A chunk of bits [pos0, end) decoded by a wave whose base (a multiple of
  // the ring) is rel0 <= pos0; a lane that is not live requests nothing.
  __host__ __device__ __forceinline__ void start(bool live, uint64_t rel0, uint64_t pos0,
                                                 uint64_t end) {
    const uint64_t b = pos0 & ~(uint64_t)(kRingBits - 1);
    const uint32_t prel = live ? (uint32_t)(pos0 - b) : 0u;
    const uint64_t len = end - b;
    off = live ? (uint32_t)((b - rel0) >> 3) : 0u;
    endr = live ? (uint32_t)(len < kMaxEnd ? len : kMaxEnd) : 0u;
    q = prel - 1;
    F = prel & ~(kSbBits - 1);
    have = F;
  }
  // The absolute bit that positions are relative to.
  __host__ __device__ __forceinline__ uint64_t base(uint64_t rel0) const {
    return rel0 + ((uint64_t)off << 3);
  }
  // The superblock at F starts within the lookahead and before the end.
  __host__ __device__ __forceinline__ bool wants() const {
    const uint32_t ahead = q + 1 + kLookaheadBits;
    return F < (ahead < endr ? ahead : endr);
  }
  // Byte of the superblock at F after the wave's base.
  __host__ __device__ __forceinline__ uint32_t load_offset() const { return off + (F >> 3); }
  __host__ __device__ __forceinline__ void requested(bool need) { F += need ? kSbBits : 0u; }
  __host__ __device__ __forceinline__ void arrived() { have = F; }
  // The ring ends before four groups' windows can.
  __host__ __device__ __forceinline__ bool low() const {
    const uint32_t reach = q + kReach;
    return have < (reach < endr ? reach : endr);
  }
  // What is in the ring and in flight ends before the windows of the four
  // groups after the next four can.
  __host__ __device__ __forceinline__ bool due() const {
    const uint32_t reach = q + kDue;
    return F < (reach < endr ? reach : endr);
  }
};

// Until no lane is low: takes what is in flight, then further superblocks
// (a low lane wants one: kReach is less than the lookahead).  W moves all
// lanes of the wave.
template <class W>
__host__ __device__ __forceinline__ void lane_reach(const LanePos& L, const W& w) {
  while (w.any(L.low())) {
    w.arrive();
    if (!w.any(L.low())) break;
    w.request();
  }
}

// Every eight groups: what was requested eight groups ago goes to the ring
// and the next superblock is requested, which keeps up with 8 bits per code.
template <class W>
__host__ __device__ __forceinline__ void lane_refill(const LanePos& L, const W& w) {
  w.arrive();
  lane_reach(L, w);
  w.request();
}

// Four groups after that: the same once more where codes run longer, so that
// their superblocks too are asked for four groups ahead.  Asked for only
// when a lane was low, each cost the wave a memory latency (1 Mi codes of 11
// bits, C = 2048: 80.9 us so, 72.8; 64 Mi uniform bytes with Table 1's
// widths 86.8, 76.2; codes of 6.7 bits unchanged).
template <class W>
__host__ __device__ __forceinline__ void lane_mid(const LanePos& L, const W& w) {
  if (w.any((int)L.low() | (int)L.due())) lane_refill(L, w);
}

// Whether a launch of the lane decoder evens out the two waves of a SIMD by
// their priority: it has to fit the device at once (two workgroups per CU),
// and with no more workgroups than CUs there is nothing to even out.  Without
// and with it, e4m3 at C = 2048 on 256 CUs: 256 workgroups 74.0 and 74.8 us,
// 260 113.7 and 108.0, 512 118.1 and 111.6; at C = 512 520 workgroups 50.5
// and 52.7, 1280 82.9 and 94.0; a batch's queue loses 7 %.  Work on another
// stream beside such a decode is not held up by it: matrix products, copies,
// small kernels and other codec calls beside five decodes ended within 2 % of
// or up to 12 % before their time without it, matrix products beside one
// decode of 2^27 symbols 8 % after.
inline bool lane_balance(uint64_t blocks, uint32_t cus) {
  return blocks > cus && blocks <= 2ull * cus;
}

}  // namespace qlc
