// The server's arena against a plain first-fit allocator, under random
// requests: blocks are placed and refused as if no spare range were lent, and
// spare ranges lie in bytes that no block and no other range holds, under the
// cap.
#include <cstdio>
#include <cstdlib>

#include "arena.hpp"

static int failures = 0;
#define EXPECT(c)                                                                   \
  do {                                                                              \
    if (!(c)) {                                                                     \
      std::fprintf(stderr, "expectation failed at line %d: %s\n", __LINE__, #c);    \
      if (++failures > 20) std::exit(1);                                            \
    }                                                                               \
  } while (0)

static uint64_t rng = 88172645463325252ull;
static uint32_t rnd(uint32_t n) {
  rng ^= rng << 13;
  rng ^= rng >> 7;
  rng ^= rng << 17;
  return uint32_t(rng >> 16) % n;
}

struct Range {
  size_t off, bytes;
};

// The first hole that holds `bytes`, between blocks sorted by offset.
static bool first_fit(const std::map<size_t, size_t>& blocks, size_t base, size_t end, size_t bytes, size_t* off) {
  size_t at = base;
  for (const auto& b : blocks) {
    if (b.first - at >= bytes) break;
    at = b.first + b.second;
  }
  *off = at;
  return end - at >= bytes;
}

int main() {
  for (int round = 0; round < 400; ++round) {
    const size_t base = 256 * rnd(5), size = 4096 + 256 * size_t(rnd(400)) + rnd(256), end = base + size;
    const size_t cap = rnd(3) ? size : size / 2;
    phg::Arena a;
    a.init(base, size, cap);
    std::map<size_t, size_t> blocks;
    std::map<uint64_t, Range> spare;
    size_t used = 0;
    uint64_t id = 0;
    for (int step = 0; step < 300; ++step) {
      ++id;
      const uint32_t what = rnd(10);
      if (what < 4) {
        const size_t bytes = 256 * (1 + size_t(rnd(uint32_t(size / 1024))));
        size_t off = 0, want = 0;
        std::vector<uint64_t> lost;
        const bool fits = used + bytes <= cap && first_fit(blocks, base, end, bytes, &want);
        const bool got = a.alloc(bytes, &off, lost);
        EXPECT(got == fits && (got || lost.empty()));
        for (uint64_t o : lost) EXPECT(spare.erase(o) == 1);
        if (got) {
          EXPECT(off == want);
          blocks[off] = bytes;
          used += bytes;
        }
      } else if (what < 6 && !blocks.empty()) {
        auto it = std::next(blocks.begin(), rnd(uint32_t(blocks.size())));
        a.release(it->first, it->second);
        used -= it->second;
        blocks.erase(it);
      } else if (what < 9) {
        const size_t bytes = 256 * (1 + size_t(rnd(8)));
        size_t off = 0;
        if (a.lend(bytes, id, &off)) {
          EXPECT(off % 256 == 0);
          spare[id] = Range{off, bytes};
        }
      } else if (!spare.empty()) {
        auto it = std::next(spare.begin(), rnd(uint32_t(spare.size())));
        a.give_back(it->second.off);
        spare.erase(it);
      }
      EXPECT(a.in_use() == used);
      size_t lent = 0;
      for (auto s = spare.begin(); s != spare.end(); ++s) {
        const Range& r = s->second;
        lent += r.bytes;
        EXPECT(r.off >= base && r.off + r.bytes <= end);
        for (const auto& b : blocks) EXPECT(r.off + r.bytes <= b.first || b.first + b.second <= r.off);
        for (auto t = std::next(s); t != spare.end(); ++t)
          EXPECT(r.off + r.bytes <= t->second.off || t->second.off + t->second.bytes <= r.off);
      }
      EXPECT(used + lent <= cap);
    }
    // all of the cap can be had as blocks, whatever is lent
    for (const auto& b : blocks) a.release(b.first, b.second);
    size_t off = 0;
    std::vector<uint64_t> lost;
    EXPECT(a.alloc(cap, &off, lost) && off == base);
  }
  // a range is lent where there is room for one
  phg::Arena a;
  a.init(0, 1024, 1024);
  size_t off = 0, s1 = 0, s2 = 0;
  std::vector<uint64_t> lost;
  EXPECT(a.alloc(512, &off, lost) && off == 0 && a.lend(256, 1, &s1) && s1 == 768 && a.lend(256, 2, &s2) && s2 == 512);
  EXPECT(!a.lend(256, 3, &s2));
  EXPECT(a.alloc(512, &off, lost) && off == 512 && lost.size() == 2);
  if (failures == 0) std::puts("all expectations held");
  return failures != 0;
}
