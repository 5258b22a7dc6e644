// Drives the list of kept device blocks without a device: sizes, limits, order.
#include <cstdio>
#include <cstdlib>
#include <vector>

#include "kept_blocks.hpp"

using namespace ann;

#define CHECK(c)                                          \
  do {                                                    \
    if (!(c)) {                                           \
      std::printf("line %d: %s\n", __LINE__, #c);         \
      std::exit(1);                                       \
    }                                                     \
  } while (0)

static void *at(size_t i) { return reinterpret_cast<void *>(i + 1); }

int main() {
  KeptBlocks kept;
  KeptBlock out[kKeepBlocks], b;
  CHECK(!kept.take_oldest(b) && !kept.take(0, 100, b));
  // the smallest that is large enough, on the right device, at most a sixteenth too large
  for (size_t i = 0; i < 4; ++i) CHECK(kept.put({at(i), (size_t)1600 + 50 * i, (int)(i == 1)}, out) == 0);
  CHECK(!kept.take(0, 1500, b));                                     // 1,600 is too large for it
  CHECK(!kept.take(2, 1600, b));
  CHECK(kept.take(0, 1590, b) && b.ptr == at(0));
  CHECK(kept.take(0, 1590, b) == false);                             // 1,700 is too large, 1,650 elsewhere
  CHECK(kept.take(0, 1650, b) && b.ptr == at(2));
  CHECK(kept.take(1, 1650, b) && b.ptr == at(1));
  CHECK(kept.count() == 1 && kept.bytes() == 1750);
  CHECK(kept.take_oldest(b) && b.ptr == at(3) && kept.count() == 0 && kept.bytes() == 0);
  // 64 blocks: the 65th sends the oldest away
  for (size_t i = 0; i < kKeepBlocks; ++i) CHECK(kept.put({at(i), 4096, 0}, out) == 0);
  CHECK(kept.put({at(64), 4096, 0}, out) == 1 && out[0].ptr == at(0) && kept.count() == kKeepBlocks);
  // 2 GiB: as many of the oldest as the newcomer needs, all of them for one of 2 GiB
  CHECK(KeptBlocks::fits(kKeepBytes) && !KeptBlocks::fits(kKeepBytes + 1));
  CHECK(kept.put({at(65), kKeepBytes - 3 * 4096, 0}, out) == kKeepBlocks - 3 && out[0].ptr == at(1));
  CHECK(kept.count() == 4 && kept.bytes() == kKeepBytes);
  CHECK(kept.put({at(66), kKeepBytes, 0}, out) == 4 && out[3].ptr == at(65) && kept.count() == 1);
  CHECK(kept.take(0, kKeepBytes, b) && b.ptr == at(66) && kept.count() == 0);
  // a request that shrinks until it fits, down to the least and no further
  for (uint64_t room : {0, 1, 127, 128, 200, 1000, 5000}) {
    uint64_t items = 3000;
    std::vector<uint64_t> asked;
    const int e = alloc_some(items, 128, [](uint64_t c) { return 8 * c; }, [&](uint64_t n) { asked.push_back(n / 8); return n / 8 <= room ? 0 : 2; }, 2);
    CHECK(e == (room < 128 ? 2 : 0) && asked.front() == 3000 && asked.back() == items && items >= 128);
    CHECK(room >= 128 || items == 128);
  }
  uint64_t items = 3000;
  CHECK(alloc_some(items, 128, [](uint64_t c) { return c; }, [](uint64_t) { return 1; }, 2) == 1 && items == 3000);   // another error: no second try
  std::printf("clean\n");
}
