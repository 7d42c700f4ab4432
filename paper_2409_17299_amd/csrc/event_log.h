// event_log.h -- the format of the lepton count pass's event log, shared by
// the kernels that write and read it (step.hip) and by a host model of both.
//
// Per wave of the count launch, a sequence of records in blocks of kLogBlock
// bytes.  A record has a fixed size, so that the reader can fetch the next
// record before it has read the current one:
//   header, 32 bytes: m_fresh (64-bit mask of the lanes that took a new
//     particle on this trip, with or without an event), m_ev (lanes with an
//     event), base (the launch index of the particle the lowest fresh lane
//     took) and tag (kLogRecord);
//   64 slots of `slot` bytes, slot l for lane l, written only for lanes with
//     an event (the event's sampled value z and its sub-interval h) or whose
//     particle, which had events, finished on this trip (its final optical
//     depth).
// The wave queue serves a trip's fresh lanes from one contiguous range, in
// lane order, so fresh lane l took particle base + (fresh lanes below l).  A
// fresh lane whose particle has no event at all finishes on that trip and is
// never replayed, but it still takes a particle: it counts in that rank.
// A block holds log_records_per_block records; the last position of a block
// is kept for a marker, a header whose tag is kLogEnd (the wave's log ends)
// or kLogJump (the log goes on in the block at offset `base`).
#pragma once

#include <stdint.h>

#if defined(__HIP__)
#define SFQED_HD __host__ __device__
#else
#define SFQED_HD
#endif

namespace sfqed {

constexpr uint64_t kLogBlock = 128 * 1024;
constexpr uint64_t kLogHeader = 32;
constexpr uint64_t kLogRecord = 0;  // tags
constexpr uint64_t kLogEnd = 1;
constexpr uint64_t kLogJump = 2;

SFQED_HD constexpr uint64_t log_record_bytes(uint32_t slot) { return kLogHeader + 64ull * slot; }
SFQED_HD constexpr uint64_t log_records_per_block(uint32_t slot) { return kLogBlock / log_record_bytes(slot); }

// What a wave with `recs` records adds to its launch's tally: the blocks it may
// take after its first one, and (from bit 40) itself, a wave with records.
constexpr uint64_t kLogTallyWave = 1ull << 40;
SFQED_HD constexpr uint64_t log_tally(uint64_t recs, uint32_t slot) {
  return recs ? kLogTallyWave + recs / (log_records_per_block(slot) - 1) : 0;
}
// Pool bytes with which a launch cannot run out, from the sum of its waves'
// tallies: when every block is handed out on demand (waves without records take
// nothing, and one block each is spare), and when the first blocks of the pool
// belong to the launch's `waves` waves, records or not.
SFQED_HD constexpr uint64_t log_need(uint64_t tally) {
  return ((tally & (kLogTallyWave - 1)) + 2 * (tally / kLogTallyWave)) * kLogBlock;
}
SFQED_HD constexpr uint64_t log_own_need(uint64_t tally, uint32_t waves) {
  return ((tally & (kLogTallyWave - 1)) + waves) * kLogBlock;
}
// Whether a launch's waves own the first blocks of a pool of `cap` bytes, which
// saves an atomic per wave on one address (50 us for 4096 waves): only where the pool holds those and
// the further blocks of every launch seen so far (own_need).  A pool that is
// smaller hands out all its blocks, so that waves without records take none.  No
// pool: the pass only measures, and needs no atomics for that.
SFQED_HD constexpr uint32_t log_own_blocks(uint64_t cap, uint64_t own_need, uint32_t waves) {
  return cap == 0 || (cap >= own_need && cap >= waves * kLogBlock) ? waves : 0;
}

// the launch index of fresh lane `lane` of a record
SFQED_HD inline uint64_t log_fresh_index(uint64_t m_fresh, uint64_t base, int lane) {
  const uint64_t below = lane == 0 ? 0ull : (m_fresh & (~0ull >> (64 - lane)));
#if defined(__HIP_DEVICE_COMPILE__)
  return base + (uint64_t)__popcll(below);
#else
  return base + (uint64_t)__builtin_popcountll(below);
#endif
}

}  // namespace sfqed
