// arena.hpp -- the server's first-fit allocator over byte offsets of its
// arena.  Plain C++, so that it also builds with an ordinary host compiler.
//
// Beside the requests' blocks it lends spare ranges: bytes that no block
// holds, for as long as none needs them.  A block is placed, and counts
// towards the cap, as if there were no spare ranges; those it overlaps, or
// that no longer fit under the cap with it, are taken back.
#pragma once

#include <stddef.h>
#include <stdint.h>

#include <iterator>
#include <map>
#include <vector>

namespace phg {

class Arena {
 public:
  void init(size_t base, size_t size, size_t cap) {
    free_.clear();
    if (size) free_[base] = size;
    cap_ = cap;
  }
  size_t in_use() const { return in_use_; }   // of blocks

  // A block of `bytes`: its offset in *off.  Owners of spare ranges that were
  // taken back for it are appended to `lost`.
  bool alloc(size_t bytes, size_t* off, std::vector<uint64_t>& lost) {
    if (in_use_ + bytes > cap_) return false;
    for (auto it = free_.begin(); it != free_.end(); ++it) {
      if (it->second < bytes) continue;
      *off = it->first;
      const size_t rem = it->second - bytes, noff = it->first + bytes;
      free_.erase(it);
      if (rem) free_[noff] = rem;
      in_use_ += bytes;
      for (auto s = spare_.begin(); s != spare_.end();) {
        const bool overlaps = s->first < *off + bytes && *off < s->first + s->second.bytes;
        if (overlaps) lost.push_back(s->second.owner);
        s = overlaps ? drop(s) : std::next(s);
      }
      while (in_use_ + spare_bytes_ > cap_) {
        lost.push_back(spare_.begin()->second.owner);
        drop(spare_.begin());
      }
      return true;
    }
    return false;
  }
  void release(size_t off, size_t bytes) {
    in_use_ -= bytes;
    auto it = free_.emplace(off, bytes).first;
    auto nx = std::next(it);
    if (nx != free_.end() && it->first + it->second == nx->first) {
      it->second += nx->second;
      free_.erase(nx);
    }
    if (it != free_.begin()) {
      auto pv = std::prev(it);
      if (pv->first + pv->second == it->first) {
        pv->second += it->second;
        free_.erase(it);
      }
    }
  }

  // A spare range of `bytes` (256-byte aligned, the highest there is) for
  // `owner`, if there are that many under the cap.
  bool lend(size_t bytes, uint64_t owner, size_t* off) {
    if (in_use_ + spare_bytes_ + bytes > cap_) return false;
    for (auto it = free_.rbegin(); it != free_.rend(); ++it) {
      size_t end = it->first + it->second;     // of the gap below the ranges seen so far
      auto s = spare_.lower_bound(end);
      for (;;) {
        const bool more = s != spare_.begin() && std::prev(s)->first >= it->first;
        const size_t begin = more ? std::prev(s)->first + std::prev(s)->second.bytes : it->first;
        if (end >= begin + bytes) {
          const size_t at = (end - bytes) & ~size_t(255);
          if (at >= begin) {
            *off = at;
            spare_[at] = Spare{bytes, owner};
            spare_bytes_ += bytes;
            return true;
          }
        }
        if (!more) break;
        --s;
        end = s->first;
      }
    }
    return false;
  }
  // The owner gives its range back (at `off`, where lend put it).
  void give_back(size_t off) {
    auto it = spare_.find(off);
    if (it != spare_.end()) drop(it);
  }

 private:
  struct Spare {
    size_t bytes;
    uint64_t owner;
  };
  std::map<size_t, size_t> free_;    // offset -> size: bytes without a block
  std::map<size_t, Spare> spare_;    // by offset; each inside one range of free_
  size_t in_use_ = 0, spare_bytes_ = 0, cap_ = 0;

  std::map<size_t, Spare>::iterator drop(std::map<size_t, Spare>::iterator it) {
    spare_bytes_ -= it->second.bytes;
    return spare_.erase(it);
  }
};

}  // namespace phg
