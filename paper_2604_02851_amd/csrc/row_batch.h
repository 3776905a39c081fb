// Rows of 32-bit words that one permutation moves through scratch memory,
// collected into batches (plain C++: also built for the CPU by the tests).
#pragma once
#include <cstdint>

namespace gs {

// Rows of one batch, all of the same length.
constexpr int kPermRows = 64;
struct RowBatch {
  uint32_t* row[kPermRows];
  int32_t count;
};

// Words from one scratch row of a batch to the next.
inline int64_t row_stride(int64_t len) { return (len + 3) / 4 * 4; }

// Hands the rows it is given to move(batch, len), in their order, as many at
// a time as the batch and scratch_words hold (at least one).  A row of length
// 0 has nothing to move and joins no batch: the moments of an empty active
// pool are 2 (11 + 3 (degree + 1)^2) such rows, more than a batch holds.
template <class Move>
class RowBatcher {
 public:
  RowBatcher(int64_t scratch_words, Move move) : scratch_words_(scratch_words), move_(move) { batch_.count = 0; }
  void add(uint32_t* row, int64_t len) {
    if (len == 0) return;
    if (len != len_) {
      flush();
      len_ = len;
    }
    batch_.row[batch_.count++] = row;
    if (batch_.count == kPermRows || (batch_.count + 1) * row_stride(len) > scratch_words_) flush();
  }
  void flush() {
    if (batch_.count > 0) move_(batch_, len_);
    batch_.count = 0;
  }

 private:
  RowBatch batch_;
  int64_t len_ = 0;
  int64_t scratch_words_;
  Move move_;
};

}  // namespace gs
