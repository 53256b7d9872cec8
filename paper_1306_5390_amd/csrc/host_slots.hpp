// host_slots.hpp -- a process-wide pool of result slots in one block of
// memory, each held by one call at a time, from any thread.  Plain C++, so that
// it also builds with an ordinary host compiler.
#pragma once

#include <stddef.h>
#include <stdint.h>

#include <mutex>

namespace phg {

class HostSlots {
 public:
  static constexpr int kSlots = 16;

  // make(bytes): the block, or null.  It is called at the first use, and again
  // at the next one after it failed (an allocation may be refused only for a
  // while); the block is kept until the process ends.
  constexpr HostSlots(size_t words, void* (*make)(size_t bytes)) : words_(words), make_(make) {}

  // Words of a slot no other call holds, or null.
  int64_t* take() {
    std::lock_guard<std::mutex> lk(mu_);
    if (block_ == nullptr) block_ = static_cast<int64_t*>(make_(sizeof(int64_t) * kSlots * words_));
    if (block_ == nullptr) return nullptr;
    for (int i = 0; i < kSlots; ++i)
      if (!used_[i]) {
        used_[i] = true;
        return block_ + size_t(i) * words_;
      }
    return nullptr;
  }
  void give_back(int64_t* slot) {
    std::lock_guard<std::mutex> lk(mu_);
    used_[size_t(slot - block_) / words_] = false;
  }

 private:
  const size_t words_;
  void* (*const make_)(size_t);
  std::mutex mu_;
  int64_t* block_ = nullptr;
  bool used_[kSlots] = {};
};

}  // namespace phg
