// Sixteen-byte loads of rows of floats that may end anywhere (k_f32_mm).  Plain C++, so that the address rule can be checked
// on the host; constexpr functions are device functions as well.
#pragma once

namespace svdmlp {

// Where to load the four floats of columns c .. c + 3 (c a multiple of four) of a row with columns 0 .. lim - 1: there, or, if
// they would pass the end of the row, its last four.  The row has room for four floats.
constexpr int row4_start(int c, int lim) {
  const int last = lim > 4 ? lim - 4 : 0;
  return c < last ? c : last;
}

// Puts what was loaded for columns c .. c + 3 into place: v[e] becomes column c + e for every such column the row has.
// Changes nothing unless c < lim < c + 4 (or c lies beyond the row).
template <class V4>
constexpr void row4_place(V4& v, int c, int lim) {
  const int s = lim > 4 ? c - (lim - 4) : 0;
  const V4 x = v;
  v[0] = s == 1 ? x[1] : s == 2 ? x[2] : s == 3 ? x[3] : x[0];
  v[1] = s == 1 ? x[2] : s == 2 ? x[3] : x[1];
  v[2] = s == 1 ? x[3] : x[2];
}

}  // namespace svdmlp
