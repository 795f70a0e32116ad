// Integer rules that the kernels follow and that the tests run on the CPU: the ranking of a token's sorted lists in calls of few
// slots, and which workgroup of the persistent FFN kernels has which units.  constexpr, and so for host and device alike.
#pragma once

#include <cstdint>

namespace sere {

// A token's top-K by ranks (ffn_small.hpp).  Key 0 is a place without an expert and belongs behind every real key, whatever that is: the
// upper half of a real key can be 0, too (an fp32 NaN whose bits are all set), and a place taken for an expert would be an index
// out of range.  So ranks go by words that are below `places` for the places without an expert, in their order, and at least `places`
// for real ones; where two words are equal, by whole keys, and by place among equal ones.
constexpr uint32_t rank_word(uint64_t key, int place, int places) {
  const uint32_t upper = static_cast<uint32_t>(key >> 32), least = static_cast<uint32_t>(places);
  if (key == 0) return least - 1 - static_cast<uint32_t>(place);
  return upper > least ? upper : least;
}
constexpr bool ranks_before(uint64_t other, int other_place, uint64_t key, int place) {
  return other > key || (other == key && other_place < place);
}

// ---- units of the persistent FFN kernels (ffn_tile.hpp).  Workgroup b is on XCD b % kXcds, the (b / kXcds)-th there (its turn).
// An XCD has places [lo, hi) of the units, of which a workgroup starts at lo + turn.
constexpr unsigned kXcds = 8;
constexpr unsigned kXcdGroups = 32;   // workgroups of an XCD

// units before XCD x's contiguous range of n
constexpr unsigned xcd_share(unsigned n, unsigned x) { return n / kXcds * x + (x < n % kXcds ? x : n % kXcds); }

// bf16: end of the whole units; the ones behind are cut into halves, one for every workgroup: places [2 whole, 2 hi).  Where at most
// half of the workgroups would get one more unit, and `pays` says so or there are no whole ones before.
constexpr unsigned whole_units_end(unsigned lo, unsigned hi, bool pays) {
  const unsigned rest = (hi - lo) % kXcdGroups;
  return rest <= kXcdGroups / 2 && (pays || rest == hi - lo) ? hi - rest : hi;
}
// Whether halves pay behind whole units.  They start a ring of their own, and a half is some two thirds of a unit: gate/up
// needs some steps for that.  A down unit stores four times the bytes, half of which is worth it at any length.  us a launch with
// halves by us without, over 170 launches of layers whose tokens select all experts, one to four whole rounds: gate/up of 1 to 3 steps
// 1.04 on average (0.98 to 1.10), 4 1.01 to 1.02, 5 and 6 0.99 (0.95 to 1.05), 7 0.99 (0.97 to 1.01), 8 to 13 0.97 (0.91 to 1.01), more
// 0.93; down of 2 to 5 steps 0.94 (0.82 to 1.00), of 7 to 13 0.96.
constexpr int kHalvesGateUpSteps = 5;
constexpr bool halves_pay(bool gate_up, int steps) { return !gate_up || steps >= kHalvesGateUpSteps; }
// first output column of place u; split: 1, or 2 for halves.  A last unit's second half may have none.
constexpr int unit_first_out(unsigned u, unsigned split, int parts, int ksplit, int out) {
  return static_cast<int>(u / split % parts / ksplit * split + u % split) * out;
}

// fp32: an XCD has an eighth of the units of the long items, which come first, and behind them an eighth of the others, counted
// from the other end.
struct LongFirst {
  unsigned longs, count;          // places of long units; of all
  unsigned to_long, to_other;     // from a place to the unit
};
constexpr LongFirst long_first(unsigned total, unsigned total_long, unsigned xcd) {
  const unsigned others = total - total_long, to_long = xcd_share(total_long, xcd), longs = xcd_share(total_long, xcd + 1) - to_long;
  const unsigned before = xcd_share(others, kXcds - xcd), after = xcd_share(others, kXcds - 1 - xcd);
  return {longs, longs + before - after, to_long, total - before - longs};
}
// The place after u: the rounds that hold long units go round the workgroups one way, the ones behind them the other way, so
// that those without a long unit get the one more that a last round has for some.
constexpr unsigned next_place_long_first(unsigned u, unsigned turn, unsigned longs) {
  const unsigned round = u / kXcdGroups + 1;
  return round * kXcdGroups + (round > longs / kXcdGroups ? kXcdGroups - 1 - turn : turn);
}
constexpr unsigned unit_at_long_first(unsigned u, unsigned longs, unsigned to_long, unsigned to_other) {
  return u + (u < longs ? to_long : to_other);
}

}  // namespace sere
