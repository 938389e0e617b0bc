// Host-side first-fit allocator over a caller-supplied device workspace.
// It hands out offsets only (the device memory itself is never touched by the
// host), is fully deterministic - the same call sequence yields the same
// offsets - and is cheap to copy, so a call can be rehearsed on a copy before
// anything is launched.
#pragma once
#include <stddef.h>

#include <map>

namespace lynx {

class Arena {
 public:
  static constexpr size_t kAlign = 256;

  explicit Arena(size_t capacity = 0) : capacity_(capacity) {
    if (capacity_ > 0) free_[0] = capacity_;
  }

  // Lowest-address block that fits; false when none does.
  bool alloc(size_t bytes, size_t* offset) {
    const size_t need = round_up(bytes == 0 ? 1 : bytes);
    for (auto it = free_.begin(); it != free_.end(); ++it) {
      if (it->second >= need) {
        const size_t off = it->first, rest = it->second - need;
        free_.erase(it);
        if (rest > 0) free_[off + need] = rest;
        used_[off] = need;
        in_use_ += need;
        if (off + need > extent_peak_) extent_peak_ = off + need;
        *offset = off;
        return true;
      }
    }
    return false;
  }

  // The block at `offset` (a multiple of kAlign); false unless all of it is free.
  bool alloc_at(size_t offset, size_t bytes) {
    const size_t need = round_up(bytes == 0 ? 1 : bytes);
    auto it = free_.upper_bound(offset);
    if (it == free_.begin()) return false;
    --it;
    const size_t first = it->first, end = it->first + it->second;
    if (offset + need > end) return false;
    free_.erase(it);
    if (offset > first) free_[first] = offset - first;
    if (end > offset + need) free_[offset + need] = end - (offset + need);
    used_[offset] = need;
    in_use_ += need;
    if (offset + need > extent_peak_) extent_peak_ = offset + need;
    return true;
  }

  // The upper end of the highest block that fits.
  bool alloc_high(size_t bytes, size_t* offset) {
    const size_t need = round_up(bytes == 0 ? 1 : bytes);
    for (auto it = free_.rbegin(); it != free_.rend(); ++it) {
      const size_t first = it->first, end = it->first + it->second;
      if (it->second < need || (end - need) / kAlign * kAlign < first) continue;
      const size_t off = (end - need) / kAlign * kAlign;
      free_.erase(first);
      if (off > first) free_[first] = off - first;
      if (end > off + need) free_[off + need] = end - (off + need);
      used_[off] = need;
      in_use_ += need;
      if (off + need > extent_peak_) extent_peak_ = off + need;
      *offset = off;
      return true;
    }
    return false;
  }

  void release(size_t offset) {
    auto u = used_.find(offset);
    if (u == used_.end()) return;
    size_t off = offset, len = u->second;
    in_use_ -= len;
    used_.erase(u);
    auto next = free_.lower_bound(off);
    if (next != free_.end() && off + len == next->first) {
      len += next->second;
      next = free_.erase(next);
    }
    if (next != free_.begin()) {
      auto prev = next;
      --prev;
      if (prev->first + prev->second == off) {
        off = prev->first;
        len += prev->second;
        free_.erase(prev);
      }
    }
    free_[off] = len;
  }

  // As if a block up to `end` had been handed out.
  void reach(size_t end) {
    if (end > extent_peak_) extent_peak_ = end;
  }

  size_t in_use() const { return in_use_; }
  size_t extent_peak() const { return extent_peak_; }  // highest byte ever handed out
  size_t capacity() const { return capacity_; }
  static size_t round_up(size_t n) { return (n + kAlign - 1) / kAlign * kAlign; }

 private:
  size_t capacity_ = 0, in_use_ = 0, extent_peak_ = 0;
  std::map<size_t, size_t> free_;  // offset -> length
  std::map<size_t, size_t> used_;  // offset -> length
};

}  // namespace lynx
