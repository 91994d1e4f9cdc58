// What ht_insert has put into a state table ht_find finds, in LDS and in memory: argument 1 is the number of
// states, argument 2 the table's bits.  Returns the number of states that are lost.
#include "wfst_lane.h"
#include <vector>

template <bool LDS> int lost(uint32_t states, int bits) {
  std::vector<wfst::Slot> table((size_t)1 << bits, wfst::Slot{~0ull, wfst::EMPTY, 0u});
  const uint32_t mask = (1u << bits) - 1u;
  int n = 0;
  for (uint32_t s = 0; s < states; ++s) {
    bool claimed = false, improved = false;
    const int at = wfst::ht_insert<LDS>(table.data(), mask, bits, 7u * s, s, claimed, improved);
    n += at < 0 || !claimed || wfst::ht_insert<LDS>(table.data(), mask, bits, 7u * s, s, claimed, improved) != at || claimed || improved;
  }
  for (uint32_t s = 0; s < states; ++s) {
    const int at = wfst::ht_find<LDS>(table.data(), mask, bits, 7u * s);
    n += at < 0 || table[(size_t)at].val != s;
  }
  return n + (states <= mask && wfst::ht_find<LDS>(table.data(), mask, bits, 7u * states) != -1);
}
int main(int, char **a) { return std::min(255, lost<true>((uint32_t)atoi(a[1]), atoi(a[2])) + lost<false>((uint32_t)atoi(a[1]), atoi(a[2]))); }
