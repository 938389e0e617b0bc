// Host-side first-fit allocator over a caller-supplied device workspace.
// It hands out offsets only (the device memory itself is never touched by the
// host), is fully deterministic - the same call sequence yields the same
// offsets - and is cheap to copy, so a call can be rehearsed on a copy before
// anything is launched.
//
// Blocks are kept in arrays of the object itself: a layer holds a few dozen at most, a pass copies its arena several times
// and places 20 to 40 blocks, and a copy of two ordered trees is an allocation per block (host side of a pass, launches
// empty, one prompt of h 5120: 6.1 us, this way 1.7, a new layer 15.2 and 4.0; a step of 256 tokens of h 256 in fp32 15.1 and 4.6).
#pragma once
#include <stddef.h>
#include <string.h>

namespace lynx {

class Arena {
 public:
  static constexpr size_t kAlign = 256;
  // 12 activations, the temporary blocks of backward (16) and the partial sums of one product are live together.
  static constexpr int kMaxBlocks = 48;

  explicit Arena(size_t capacity = 0) : capacity_(capacity) {
    if (capacity_ > 0) free_[n_free_++] = {0, capacity_};
  }
  Arena(const Arena& o) { *this = o; }
  Arena& operator=(const Arena& o) {
    if (this == &o) return *this;
    capacity_ = o.capacity_;
    in_use_ = o.in_use_;
    extent_peak_ = o.extent_peak_;
    n_free_ = o.n_free_;
    n_used_ = o.n_used_;
    memcpy(free_, o.free_, sizeof(Block) * static_cast<size_t>(n_free_));
    memcpy(used_, o.used_, sizeof(Block) * static_cast<size_t>(n_used_));
    return *this;
  }

  // Lowest-address block that fits; false when none does.
  bool alloc(size_t bytes, size_t* offset) {
    const size_t need = round_up(bytes == 0 ? 1 : bytes);
    for (int i = 0; i < n_free_; ++i)
      if (free_[i].len >= need) return take(i, free_[i].off, need, offset);
    return false;
  }

  // The block at `offset` (a multiple of kAlign); false unless all of it is free.
  bool alloc_at(size_t offset, size_t bytes) {
    const size_t need = round_up(bytes == 0 ? 1 : bytes);
    const int i = after(offset) - 1;
    return i >= 0 && offset + need <= free_[i].off + free_[i].len && take(i, offset, need, &offset);
  }

  // The upper end of the highest block that fits.
  bool alloc_high(size_t bytes, size_t* offset) {
    const size_t need = round_up(bytes == 0 ? 1 : bytes);
    for (int i = n_free_ - 1; i >= 0; --i) {
      if (free_[i].len < need) continue;
      const size_t off = (free_[i].off + free_[i].len - need) / kAlign * kAlign;
      if (off >= free_[i].off) return take(i, off, need, offset);
    }
    return false;
  }

  void release(size_t offset) {
    int u = 0;
    while (u < n_used_ && used_[u].off != offset) ++u;
    if (u == n_used_) return;
    const Block b = used_[u];
    used_[u] = used_[--n_used_];
    in_use_ -= b.len;
    const int next = after(b.off);
    const bool joins_prev = next > 0 && free_[next - 1].off + free_[next - 1].len == b.off;
    const bool joins_next = next < n_free_ && b.off + b.len == free_[next].off;
    if (joins_prev) {
      free_[next - 1].len += b.len;
      if (joins_next) {
        free_[next - 1].len += free_[next].len;
        erase(next);
      }
    } else if (joins_next) {
      free_[next] = {b.off, b.len + free_[next].len};
    } else {
      insert(next, b);
    }
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
  struct Block { size_t off, len; };

  // Index of the first free block beyond `offset`.
  int after(size_t offset) const {
    int i = 0;
    while (i < n_free_ && free_[i].off <= offset) ++i;
    return i;
  }
  void erase(int i) {
    --n_free_;
    memmove(free_ + i, free_ + i + 1, sizeof(Block) * static_cast<size_t>(n_free_ - i));
  }
  void insert(int i, Block b) {
    memmove(free_ + i + 1, free_ + i, sizeof(Block) * static_cast<size_t>(n_free_ - i));
    ++n_free_;
    free_[i] = b;
  }
  // `need` bytes at `off` out of free block i.
  bool take(int i, size_t off, size_t need, size_t* offset) {
    if (n_used_ == kMaxBlocks) return false;
    const Block b = free_[i];
    const size_t end = off + need, b_end = b.off + b.len;
    if (off > b.off) {
      free_[i].len = off - b.off;
      if (b_end > end) insert(i + 1, {end, b_end - end});
    } else if (b_end > end) {
      free_[i] = {end, b_end - end};
    } else {
      erase(i);
    }
    used_[n_used_++] = {off, need};
    in_use_ += need;
    reach(end);
    *offset = off;
    return true;
  }

  size_t capacity_ = 0, in_use_ = 0, extent_peak_ = 0;
  int n_free_ = 0, n_used_ = 0;
  Block free_[kMaxBlocks + 1];  // by offset; no two touch, so at most one more than there are blocks in use
  Block used_[kMaxBlocks];      // in no order
};

}  // namespace lynx
