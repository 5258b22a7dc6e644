// Multi-expansion search kernels for small batches, eight expansions per step (see search_relay.hpp).
#include "search_relay.hpp"

namespace ann {
ann_status launch_search_relay_wide(const SearchArgs &a, uint32_t bits, uint32_t lpr, int m, hipStream_t st) {
  return bits == 8 ? launch_relay<8, kMaxExpansionsPerStep>(a, lpr, m, st) : launch_relay<4, kMaxExpansionsPerStep>(a, lpr, m, st);
}
}  // namespace ann
