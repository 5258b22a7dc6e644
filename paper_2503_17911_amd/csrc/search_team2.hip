// Search kernels with two wavefronts per query (see search_kernel.hpp).
#include "search_kernel.hpp"

namespace ann {
ann_status launch_search_team2(const SearchArgs &a, uint32_t bits, uint32_t lpr, int m, bool wide_step, hipStream_t st) {
  return launch_team<2>(a, bits, lpr, m, wide_step, st);
}
}  // namespace ann
