// One-expansion search kernels for small batches (see search_kernel.hpp).
#include "search_kernel.hpp"

namespace ann {
ann_status launch_search_small(const SearchArgs &a, uint32_t bits, uint32_t lpr, int m, hipStream_t st) {
  return bits == 8 ? launch_small<8>(a, lpr, m, st) : launch_small<4>(a, lpr, m, st);
}
}  // namespace ann
