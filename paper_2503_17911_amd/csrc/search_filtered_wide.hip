// Search kernels with the edge filter, up to eight expansions per step (see search_kernel.hpp).
#include "search_kernel.hpp"

namespace ann {
ann_status launch_search_filtered_wide(const SearchArgs &a, uint32_t bits, uint32_t lpr, int m, hipStream_t st) {
  return launch_search<false, true, true>(a, bits, lpr, m, true, st);
}
}  // namespace ann
