// One-expansion filtered search kernels for small batches (see search_chain.hpp).
#include "search_chain.hpp"

namespace ann {
ann_status launch_search_chain_filtered(const SearchArgs &a, uint32_t bits, uint32_t lpr, int m, hipStream_t st) {
  return bits == 8 ? launch_chain<8, true>(a, lpr, m, st) : launch_chain<4, true>(a, lpr, m, st);
}
}  // namespace ann
