// What the product's activation loaders may read of X (plain C++: the host
// checks it too).
#pragma once

#include <cstdint>

namespace ojbkq {

// Whether the eight elements from X[r][t] on (r < m, t < T; rows of T elements
// at a stride ldx >= T) can be read as one piece: it ends inside its row, or
// reads on into the row after it.  The row stride is at least T, so from T = 8
// on one further row holds the at most seven elements past the row's end;
// shorter rows need not (m x 1 contiguous: row m - 2 has two elements left).
constexpr bool x_piece_inside(int64_t r, int64_t t, int64_t m, int64_t T) {
  return t + 8 <= T || (T >= 8 && r + 1 < m);
}

}  // namespace ojbkq
