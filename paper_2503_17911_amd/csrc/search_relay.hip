// Multi-expansion search kernels for small batches (see search_relay.hpp).
#include "search_relay.hpp"

namespace ann {
ann_status launch_search_relay_wide(const SearchArgs &a, uint32_t bits, uint32_t lpr, int m, hipStream_t st);
ann_status launch_search_relay(const SearchArgs &a, uint32_t bits, uint32_t lpr, int m, bool wide_step, hipStream_t st) {
  if (wide_step) return launch_search_relay_wide(a, bits, lpr, m, st);
  return bits == 8 ? launch_relay<8, kDefaultExpansionsPerStep>(a, lpr, m, st) : launch_relay<4, kDefaultExpansionsPerStep>(a, lpr, m, st);
}
}  // namespace ann
