// State and protocol of the grid barrier, without the device code around it
// (`grid_barrier` in iwpp_device.hpp), so that a host program can run it too.
//
// Workgroup b counts itself in group b mod 8's counter: its low half counts the
// arrivals (they only grow: number (gen + 1) * size is generation gen's last),
// its high half the list items the group's workgroups have appended.  The last
// arrival of a group at generation gen writes the group's word, the items and
// gen + 1; a workgroup leaves when the words of all groups say gen + 1.
//
// A group that has left a barrier may reach the next one, and its last arrival
// there write the group's word, while a workgroup of another group is still
// polling the first.  So consecutive generations use two words in turn: the word
// of generation gen is written again for generation gen + 2, which needs every
// workgroup to have arrived at gen + 1 and so to have left gen.  Until then it
// says exactly gen + 1 beside exactly the items appended before the barrier.
// (With one word a group the late poller would pass on a word of the generation
// after, take items of the next round for this round's, and miss them then.)
#pragma once

#include <stdint.h>

namespace iwpp {

struct GridBarrier {
  unsigned long long group[8][32];  // 256 bytes apart: no two counters share a cache line
  unsigned long long word[2][8];    // by generation parity; one cache line
  unsigned long long pad[16];
  uint32_t abort[64];
};

namespace barrier {

// What an arrival adds to its group's counter.
constexpr unsigned long long arrival(uint32_t items) { return (unsigned long long)items << 32 | 1ull; }
// Is the arrival that made the counter `total` its group's last at generation gen?
constexpr bool last(unsigned long long total, uint32_t gen, uint32_t in_group) {
  return (uint32_t)total == (gen + 1u) * in_group;
}
// Which of a group's words generation gen uses, what its last arrival writes, and
// whether a word read is that.
constexpr uint32_t slot(uint32_t gen) { return (gen + 1u) & 1u; }
constexpr unsigned long long word(unsigned long long total, uint32_t gen) {
  return (total & ~0xFFFFFFFFull) | (gen + 1u);
}
constexpr bool arrived(unsigned long long v, uint32_t gen) { return (uint32_t)v == gen + 1u; }
// Items the group has appended up to the word's barrier (modulo 2^32).
constexpr uint32_t items(unsigned long long v) { return (uint32_t)(v >> 32); }

}  // namespace barrier
}  // namespace iwpp
