// The parts of the one-sided Jacobi (row_sweep.h) that are plain functions of numbers, so that a host compiler
// takes them too.
#pragma once

namespace gipeps {

// Where the column scales (d, 1/d) lie in LDS, in entries of two doubles, for ng column groups.  Three ranges
// that share no entry:
//   lower(k)  the scales of group k's first column, which group k - 1 reads between the two barriers of a
//             boundary round;
//   upper(k)  those of the column that group k hands up, which group k + 1 reads after the second barrier;
//   end(p)    at the end of a sweep, the scales of slots 2 p and 2 p + 1, for the J rows.
// No barrier lies between a sweep's last read of upper and its first write of end, and reader and writer are
// in different waves from 33 columns on: with end over lower and upper, a group of four columns, which writes
// two entries of end, could overwrite an entry of upper that another wave had still to read.
struct JacobiScales {
  int ng;
  constexpr int lower(int k) const { return k; }
  constexpr int upper(int k) const { return ng + k; }
  constexpr int end(int p) const { return 2 * ng + p; }
  // entries for up to maxn columns in groups of nc
  static constexpr int room(int maxn, int nc) { return 2 * (maxn / nc) + maxn / 2; }
};

}  // namespace gipeps
