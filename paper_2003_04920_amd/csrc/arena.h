// Device memory of one handle.  A handle keeps some forty arrays, most of them small, and
// every hipFree costs 100 to 450 us whatever its size: destroying the two handles of a
// 200,000-vertex layout took 5.0 ms of its 18, now 1.7 of 11, and a growing planner paid for
// every array it replaced.  Here pieces come from a few slabs that go back to the device with
// the handle.
//
// A freed piece is used again by the same handle only, and all of a handle's work is on its
// one stream, so a new user is ordered after the old one without a wait.  Requests past
// kDirect get memory of their own and give it back when freed: graphs near the size of the
// device's memory find as much of it as before.  Not thread-safe, as the handles are not.
#pragma once

#include <hip/hip_runtime.h>

#include <algorithm>
#include <map>
#include <vector>

namespace pirrt {

class Arena {
 public:
  static constexpr size_t kAlign = 256;
  static constexpr size_t kFirst = (size_t)1 << 20;
  static constexpr size_t kDirect = (size_t)128 << 20;
  static constexpr size_t kSlabMax = (size_t)256 << 20;  // of a slab that was foreseen (expect)
  static constexpr size_t kGrow = (size_t)64 << 20;      // of the others

  Arena() = default;
  Arena(const Arena&) = delete;
  Arena& operator=(const Arena&) = delete;
  ~Arena() { release(); }

  // nullptr if the device (or the host, for the books) has no room.
  void* alloc(size_t bytes) {
    bytes = (std::max(bytes, (size_t)1) + kAlign - 1) / kAlign * kAlign;
    if (bytes > kDirect) return device(bytes);
    try {
      auto best = free_.end();
      for (auto it = free_.begin(); it != free_.end(); ++it)
        if (it->second >= bytes && (best == free_.end() || it->second < best->second)) best = it;
      if (best == free_.end()) {
        // slabs grow with the handle, so that their number stays small, but not far past what
        // is asked for: the driver wipes all of them when they go back
        size_t size = std::max({bytes, std::min(std::max(2 * total_, kFirst), kGrow), std::min(expected_, kSlabMax)});
        expected_ = 0;
        slabs_.reserve(slabs_.size() + 1);
        char* p = static_cast<char*>(device(size));
        if (!p && size > bytes) p = static_cast<char*>(device(size = bytes));
        if (!p) return nullptr;
        slabs_.push_back(p);
        total_ += size;
        best = free_.emplace(p, size).first;
      }
      char* p = best->first;
      const size_t rest = best->second - bytes;
      used_[p] = bytes;
      free_.erase(best);
      if (rest) free_[p + bytes] = rest;
      return p;
    } catch (...) {
      return nullptr;
    }
  }

  // About this many bytes will be asked for soon: the next slab holds them.
  void expect(size_t bytes) { expected_ = bytes; }

  void free(void* ptr) {
    if (!ptr) return;
    char* p = static_cast<char*>(ptr);
    auto u = used_.find(p);
    if (u == used_.end()) {
      (void)hipFree(ptr);
      return;
    }
    size_t size = u->second;
    used_.erase(u);
    try {
      auto next = free_.lower_bound(p);
      // (pieces of two slabs are joined only where the slabs are neighbours by chance: apart)
      if (next != free_.end() && p + size == next->first && !starts_slab(next->first)) {
        size += next->second;
        next = free_.erase(next);
      }
      if (next != free_.begin() && !starts_slab(p)) {
        auto prev = std::prev(next);
        if (prev->first + prev->second == p) {
          prev->second += size;
          return;
        }
      }
      free_[p] = size;
    } catch (...) {  // the piece is out of use until the handle goes
    }
  }

  void release() {
    for (char* s : slabs_) (void)hipFree(s);
    slabs_.clear();
    free_.clear();
    used_.clear();
    total_ = 0;
  }

 private:
  static void* device(size_t bytes) {
    void* p = nullptr;
    if (hipMalloc(&p, bytes) != hipSuccess) {
      (void)hipGetLastError();
      return nullptr;
    }
    return p;
  }
  bool starts_slab(char* p) const { return std::find(slabs_.begin(), slabs_.end(), p) != slabs_.end(); }

  std::vector<char*> slabs_;
  std::map<char*, size_t> free_, used_;  // pieces by address
  size_t total_ = 0, expected_ = 0;
};

}  // namespace pirrt
