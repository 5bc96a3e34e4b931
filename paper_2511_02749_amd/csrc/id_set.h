// A set of ids in [0, n) as a bitmap under levels of summary bitmaps (a bit per word of the
// level below, up to a single word): the lowest member, an insertion and a removal each touch
// at most a word per level (four levels for 16 million ids, six for 2^31).
#pragma once
#include <cstddef>
#include <cstdint>
#include <vector>

namespace spanq {

class IdSet {
 public:
  void resize(int64_t n) {  // empty, of ids in [0, n)
    levels_.clear();
    size_t words = static_cast<size_t>(n);
    do {
      words = (words + 63) / 64;
      levels_.emplace_back(words, 0);
    } while (words > 1);
    size_ = 0;
  }
  bool empty() const { return size_ == 0; }
  int64_t size() const { return size_; }
  bool contains(int64_t i) const { return (levels_[0][i >> 6] >> (i & 63)) & 1; }
  void insert(int64_t i) {  // not a member yet
    for (auto& level : levels_) {
      uint64_t& w = level[i >> 6];
      const bool summarised = w != 0;
      w |= uint64_t{1} << (i & 63);
      if (summarised) break;
      i >>= 6;
    }
    ++size_;
  }
  void erase(int64_t i) {  // a member
    for (auto& level : levels_) {
      if ((level[i >> 6] &= ~(uint64_t{1} << (i & 63))) != 0) break;
      i >>= 6;
    }
    --size_;
  }
  int32_t lowest() const {  // of a set that is not empty
    size_t at = 0;
    for (size_t l = levels_.size(); l-- > 0;) at = 64 * at + static_cast<size_t>(__builtin_ctzll(levels_[l][at]));
    return static_cast<int32_t>(at);
  }
  void clear() {  // one member at a time while they are fewer than the words
    if (size_ < static_cast<int64_t>(levels_[0].size()))
      while (!empty()) erase(lowest());
    else
      for (auto& level : levels_) level.assign(level.size(), 0);
    size_ = 0;
  }

 private:
  std::vector<std::vector<uint64_t>> levels_;
  int64_t size_ = 0;
};

}  // namespace spanq
