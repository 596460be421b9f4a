// Row and column of the entries of a dense row-major matrix as a group of threads walks them.
#pragma once

namespace subadmm {

// Thread `rank` of `size` takes entries rank, rank + size, ... of rows of n entries.  The row and
// column follow by carry from two integer divisions at the start, so they are exact for every
// matrix whose entries an int counts, and an entry costs an add and a select (a quotient formed
// in FP32 per entry was off by one from 4.2 million entries on).  constexpr: used on the host too.
struct RowWalk {
  int row, col;      // of the current entry
  int drow, dcol;    // size / n and its remainder
  int n;
  constexpr RowWalk(int rank, int size, int n_)
      : row(rank / n_), col(rank % n_), drow(size / n_), dcol(size % n_), n(n_) {}
  constexpr void next() {
    row += drow;
    col += dcol;
    if (col >= n) {
      col -= n;
      ++row;
    }
  }
};

}  // namespace subadmm
