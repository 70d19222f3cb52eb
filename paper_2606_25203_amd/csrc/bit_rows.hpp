// bit_rows.hpp -- host arithmetic of the bit-packed sweeps' rows (bits.hip):
// which graphs have them, and where they start.  Plain C++, no device code.
#pragma once
#include <stdint.h>
#include <stdlib.h>

#include <vector>

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

// The rows of a graph (rp, col, J: internal ids): an entry is the byte offset of
// the neighbour's mask in a group of one tile, of its complement along negative
// couplings where there are both; the higher neighbours come first (the edges
// of the energy sum), then the lower, then the mask that is always 0 up to a
// multiple of 4 (with a stride, to the next row).  brows: per vertex (np of
// them) its bounds, then the table offset of a count of 0, then the number of
// higher neighbours.
inline void fill_bit_rows(int32_t n, const int32_t* rp, const int32_t* col, const int32_t* J, bool both,
                          int32_t maxdeg, int32_t stride, int64_t padded, std::vector<int32_t>& brows,
                          std::vector<int32_t>& bent) {
  const int32_t np = (n + 3) & ~3;
  brows.assign((size_t)np * 4, 0);
  bent.assign((size_t)bit_row_entries(n, stride, padded), 8 * np);
  int32_t *bounds = brows.data(), *base = bounds + 2 * (size_t)np, *higher = base + np;
  int32_t at = 0;
  for (int32_t v = 0; v < np; ++v) {
    if (stride) at = v * stride;
    bounds[2 * v] = bounds[2 * v + 1] = at;
    if (v >= n) continue;
    const int32_t e0 = rp[v], deg = rp[v + 1] - e0;
    int32_t* const row = bent.data() + at;
    int32_t up = 0, low = deg;
    for (int32_t e = e0; e < e0 + deg; ++e) {  // (no branch: the order of neighbours is random)
      const bool above = col[e] > v;
      low -= !above;
      row[above ? up : low] = 8 * (col[e] + (both && J[e] < 0 ? np + 1 : 0));
      up += above;
    }
    at += (deg + 3) & ~3;
    bounds[2 * v + 1] = at;
    base[v] = 4 * (maxdeg - deg);
    higher[v] = up;
  }
}

// How a graph of couplings of one magnitude keeps its fields when its longest
// row is far longer than the others: one wavefront walks a row, so a phase then
// lasts as long as that row whatever else it does.
enum class LongRows { kBits, kGathered, kAsOthers };

// Rows of more than 128 entries and more than 8 times the average are long
// (none: kBits).  With them a population of at most two tiles, or of fewer than
// 2^20 spins, is as long as its rows' chains in any form but incremental fields
// (kAsOthers: what graphs of several magnitudes take); up to 2^24 spins gathering
// shares the row's entries among the tiles of a wave, four with few masks in
// flight do not; above that all rows together take longer.  From 16 neighbours
// on average the other rows weigh more: bit-packed also below 2^20 (up to two
// tiles) and 2^22 spins.  Runs of 20 steps of 1 (3) sweeps up to beta 4, fields
// kept, gathered, bit-packed, ms; heavy-tailed degrees up to 256, average 8:
// n = 3,000, R = 64: 1.35 (2.5), 1.64 (3.4), 1.73 (2.9); R = 1,024: 1.73 (3.4),
// 1.58 (3.1), 2.49 (4.1); n = 20,000, R = 64: 1.67 (3.3), 2.04 (4.4), 2.31 (4.0);
// R = 256: 2.27 (4.7), 2.11 (4.5), 3.51 (6.2); R = 1,024: 4.33 (10.2), 3.42 (8.2),
// 4.29 (7.7).  Average 20: n = 3,000, R = 512: 2.12 (4.5), 2.51 (6.1), 2.39 (4.8);
// n = 20,000, R = 256: 3.11 (7.0), 3.63 (7.9), 5.19 (10.1).  Average 34, R = 512,
// n = 20,000: 5.68 (14.2), 6.40 (17.0), 6.60 (13.3).  Up to beta 1, where flips
// are many: average 8, n = 20,000, R = 256: 3.18 (7.7), 2.30 (5.1), 3.54 (6.3);
// average 20: 4.54 (12.0), 3.70 (8.4), 5.18 (10.1), n = 3,000, R = 512: 2.61 (6.2),
// 2.54 (6.2), 2.42 (4.9).  A graph whose only rows
// above 64 are one or two keeps those rows' fields in either form (kAsOthers).
inline LongRows long_row_form(int64_t n, int64_t entries, int64_t maxdeg, int64_t above64, int64_t tiles) {
  if (maxdeg <= 128 || maxdeg * n <= 8 * entries) return LongRows::kBits;
  const bool few = entries < 16 * n;
  const int64_t spins = 64 * n * tiles, million = 1 << 20;
  if (tiles <= 2 ? few || spins >= million : few && spins < million) return LongRows::kAsOthers;
  if (tiles <= 2 || spins < (few ? 1 : 4) * million || spins >= 16 * million) return LongRows::kBits;
  return above64 <= 2 ? LongRows::kAsOthers : LongRows::kGathered;
}

}  // namespace pamc
