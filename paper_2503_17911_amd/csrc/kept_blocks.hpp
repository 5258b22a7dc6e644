// Which freed blocks of device memory are kept for the next request (host.hip),
// without the allocator behind it: host code that a CPU test can drive.
#pragma once
#include <stddef.h>
#include <stdint.h>

namespace ann {

struct KeptBlock {
  void *ptr = nullptr;
  size_t bytes = 0;
  int device = 0;
};

constexpr int kKeepBlocks = 64;
constexpr size_t kKeepBytes = (size_t)2 << 30;

// At most kKeepBlocks blocks and kKeepBytes bytes, oldest first.
class KeptBlocks {
 public:
  // The smallest kept block on the device that holds `want` bytes and is at most
  // a sixteenth larger (an index keeps what it is given for its whole life).
  bool take(int device, size_t want, KeptBlock &out) {
    int best = -1;
    for (int i = 0; i < n_; ++i)
      if (block_[i].device == device && block_[i].bytes >= want && block_[i].bytes - want <= want / 16 &&
          (best < 0 || block_[i].bytes < block_[best].bytes))
        best = i;
    return best >= 0 && remove(best, out);
  }
  // The block kept longest.
  bool take_oldest(KeptBlock &out) { return n_ > 0 && remove(0, out); }
  // Whether a block of this size is kept at all.
  static bool fits(size_t bytes) { return bytes <= kKeepBytes; }
  // Keeps a block that fits; returns how many were put into `out` to make room for it.
  int put(const KeptBlock &b, KeptBlock (&out)[kKeepBlocks]) {
    int n_out = 0;
    while (n_ == kKeepBlocks || bytes_ + b.bytes > kKeepBytes) remove(0, out[n_out++]);
    block_[n_++] = b;
    bytes_ += b.bytes;
    return n_out;
  }
  int count() const { return n_; }
  size_t bytes() const { return bytes_; }

 private:
  bool remove(int i, KeptBlock &out) {
    out = block_[i];
    for (int j = i; j + 1 < n_; ++j) block_[j] = block_[j + 1];
    --n_;
    bytes_ -= out.bytes;
    return true;
  }
  KeptBlock block_[kKeepBlocks];
  int n_ = 0;
  size_t bytes_ = 0;
};

// alloc(bytes(items)) or, as long as that returns `no_memory`, the same for half as many items down to `least`.
template <typename Bytes, typename Alloc, typename Status>
Status alloc_some(uint64_t &items, uint64_t least, Bytes bytes, Alloc alloc, Status no_memory) {
  for (;;) {
    const Status e = alloc(bytes(items));
    if (e != no_memory || items <= least) return e;
    items = items / 2 > least ? items / 2 : least;
  }
}

}  // namespace ann
