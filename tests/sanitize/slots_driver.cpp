// The pool of result slots: a refused block is asked for again, a slot is held
// by one call at a time, and none is handed out beyond the last.
#include <cstdio>
#include <cstdlib>
#include <set>
#include <thread>
#include <vector>

#include "host_slots.hpp"

static int failures = 0;
#define EXPECT(c)                                                                \
  do {                                                                           \
    if (!(c)) {                                                                  \
      std::fprintf(stderr, "expectation failed at line %d: %s\n", __LINE__, #c); \
      ++failures;                                                                \
    }                                                                            \
  } while (0)

static int asked = 0, refuse = 2;
static std::vector<int64_t> block;
static void* make(size_t bytes) {
  ++asked;
  if (refuse-- > 0) return nullptr;
  block.resize(bytes / sizeof(int64_t));
  return block.data();
}

static phg::HostSlots slots(100, make);

int main() {
  EXPECT(slots.take() == nullptr && slots.take() == nullptr && asked == 2);
  std::set<int64_t*> got;
  for (int i = 0; i < phg::HostSlots::kSlots; ++i) {
    int64_t* s = slots.take();
    EXPECT(s != nullptr && got.insert(s).second);
    if (s != nullptr) s[0] = s[99] = i;
  }
  EXPECT(asked == 3 && slots.take() == nullptr);
  for (int64_t* s : got) slots.give_back(s);
  // many threads: a slot's words are its holder's
  std::vector<std::thread> threads;
  int mixed[24] = {};
  for (int t = 0; t < 24; ++t)
    threads.emplace_back([t, &mixed] {
      for (int i = 0; i < 2000; ++i) {
        int64_t* s = slots.take();
        if (s == nullptr) continue;
        s[0] = s[99] = t;
        std::this_thread::yield();
        if (s[0] != t || s[99] != t) ++mixed[t];
        slots.give_back(s);
      }
    });
  for (auto& t : threads) t.join();
  for (int m : mixed) EXPECT(m == 0);
  EXPECT(asked == 3);
  if (failures == 0) std::puts("all expectations held");
  return failures != 0;
}
