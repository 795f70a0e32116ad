// Integer rules that the kernels follow and that the tests run on the CPU: the ranking of a token's sorted lists in calls of few
// slots.  constexpr, and so for host and device alike.
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

}  // namespace sere
