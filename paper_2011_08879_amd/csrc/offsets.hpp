// Walks through ranges of entry offsets.
#pragma once

#include <cstdint>

namespace gko {

// Offsets b + first, b + first + S, ... of the range [b, e).  A matrix holds up
// to 2^31 - 2 entries, so near its end the offset of the step past a range may
// not fit int32: what is left of the range is counted instead, which always
// does.  at() is an offset of the range while more() holds; left() counts the
// entries from there to the range's end.
template <int32_t S>
class entry_steps {
  public:
    constexpr entry_steps(int32_t b, int32_t e, int32_t first = 0) : e_(e), left_(e - b - first) {}
    constexpr bool more() const { return left_ > 0; }
    constexpr void next() { left_ -= S; }
    constexpr int32_t at() const { return e_ - left_; }
    constexpr int32_t left() const { return left_; }
    // the entries of this step
    constexpr int32_t count() const { return left_ < S ? left_ : S; }

  private:
    int32_t e_, left_;
};

}  // namespace gko
