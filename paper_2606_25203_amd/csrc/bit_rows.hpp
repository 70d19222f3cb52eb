// bit_rows.hpp -- host arithmetic of the bit-packed sweeps' rows (bits.hip):
// which graphs have them, and where they start.  Plain C++, no device code.
#pragma once
#include <stdint.h>
#include <stdlib.h>

namespace pamc {

// Longest row of a bit-packed instance: one wavefront walks a row, and the
// threshold table (4 deg + 4 entries) is staged in LDS by every work-group.
constexpr int32_t kBitsMaxDegree = 256;

// Entries after the last row: kernels read up to 16 from a row's start, and
// with a stride from those of a whole quad.
inline int64_t bit_row_tail(int64_t stride) { return 16 + 4 * stride; }

// Row stride (0: rows follow each other) of n rows (np with the padding
// vertices), the longest of maxdeg entries, `padded` in all when each is padded
// to a multiple of 4.  Rows start at multiples of one stride where that costs
// at most three times the entries: a wave then finds its row without reading
// bounds.  Kernels and row bounds count entries in 32 bits.
inline int32_t bit_row_stride(int64_t n, int64_t maxdeg, int64_t padded) {
  const int64_t stride = (maxdeg + 3) & ~(int64_t)3, np = (n + 3) & ~(int64_t)3;
  return stride * n <= 3 * padded && stride * np + bit_row_tail(stride) <= INT32_MAX ? (int32_t)stride : 0;
}

// Whether the rows can be counted in 32 bits at all.
inline bool bit_rows_fit(int64_t padded) { return padded + bit_row_tail(0) <= INT32_MAX; }

// Entries of the rows, the tail included.
inline int64_t bit_row_entries(int64_t n, int64_t stride, int64_t padded) {
  return (stride ? stride * ((n + 3) & ~(int64_t)3) : padded) + bit_row_tail(stride);
}

// The magnitude of a graph whose couplings all have one, whose rows have at
// most kBitsMaxDegree entries and whose padded rows (*padded entries) fit 32
// bits; else 0.  *both: couplings of both signs.
inline int32_t one_magnitude(int32_t n, const int32_t* rp, const int32_t* J, bool* both, int64_t* padded) {
  *both = false;
  *padded = 0;
  if (rp[n] == 0 || n > (1 << 24) || J[0] == INT32_MIN) return 0;
  const int32_t c = abs(J[0]);
  for (int32_t v = 0; v < n; ++v) {
    const int32_t deg = rp[v + 1] - rp[v];
    if (deg > kBitsMaxDegree) return 0;
    *padded += (deg + 3) & ~3;
  }
  if (!bit_rows_fit(*padded)) return 0;
  for (int32_t e = 0; e < rp[n]; ++e) {
    if (J[e] != c && J[e] != -c) return 0;
    if (J[e] != J[0]) *both = true;
  }
  return c;
}

}  // namespace pamc
