"""Host arithmetic of the bit-packed sweeps' rows (csrc/bit_rows.hpp), built
with the host compiler: kernels and row bounds count entries in 32 bits, so
graphs whose rows would need more of them, with a stride or at all, are told
apart from those that fit."""
import os
import subprocess

import numpy as np
import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2606_25203_amd", "csrc")
INT32_MAX = 2**31 - 1

PROGRAM = r"""
#include "bit_rows.hpp"
#include <stdio.h>
#include <vector>
int main() {
  char what;
  long long a, b, c, d;
  while (scanf(" %c %lld %lld %lld", &what, &a, &b, &c) == 4) {
    if (what == 'f') {  // form of n rows, b entries in all, the longest of c, d tiles
      if (scanf(" %lld", &d) != 1) return 1;
      for (int above64 : {2, 3}) printf("%d ", (int)pamc::long_row_form(a, b, c, above64, d));
      printf("\n");
    } else if (what == 'r') {  // rows of a graph of a vertices, b entries; c: couplings of both signs; d: stride or not
      if (scanf(" %lld", &d) != 1) return 1;
      std::vector<int32_t> rp(a + 1), col(b), J(b), brows, bent;
      for (auto* x : {&rp, &col, &J})
        for (int32_t& y : *x)
          if (scanf(" %d", &y) != 1) return 1;
      int32_t maxdeg = 0;
      int64_t padded = 0;
      for (long long v = 0; v < a; ++v) {
        const int32_t deg = rp[v + 1] - rp[v];
        maxdeg = deg > maxdeg ? deg : maxdeg;
        padded += (deg + 3) & ~3;
      }
      const int32_t stride = d ? (maxdeg + 3) & ~3 : 0;
      pamc::fill_bit_rows((int32_t)a, rp.data(), col.data(), J.data(), c != 0, maxdeg, stride, padded, brows, bent);
      printf("%d %zu", stride, brows.size());
      for (int32_t x : brows) printf(" %d", x);
      for (int32_t x : bent) printf(" %d", x);
      printf("\n");
    } else if (what == 's') {  // stride of n rows, and the entries with it
      const int32_t s = pamc::bit_row_stride(a, b, c);
      printf("%d %lld %d\n", s, (long long)pamc::bit_row_entries(a, s, c), (int)pamc::bit_rows_fit(c));
    } else {  // n rows of b entries each: the entries themselves are not read before the rows are counted
      std::vector<int32_t> rp(a + 1);
      for (long long v = 0; v <= a; ++v) rp[v] = (int32_t)(v * b);
      std::vector<int32_t> J(c, 3);
      bool both;
      int64_t padded;
      const int32_t m = pamc::one_magnitude((int32_t)a, rp.data(), J.data(), &both, &padded);
      printf("%d %d %lld\n", m, (int)both, (long long)padded);
    }
  }
}
"""


@pytest.fixture(scope="module")
def ask(tmp_path_factory):
    d = tmp_path_factory.mktemp("bit_rows")
    (d / "rows.cpp").write_text(PROGRAM)
    exe = str(d / "rows")
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-fsanitize=undefined", "-fno-sanitize-recover",
                    "-I", CSRC, str(d / "rows.cpp"), "-o", exe], check=True)

    def run(what, *args):
        out = subprocess.run([exe], input=" ".join(map(str, (what, *args))) + "\n", capture_output=True, text=True, check=True).stdout
        return [int(x) for x in out.split()]
    return run


@pytest.mark.parametrize("n,maxdeg,padded,stride", [
    (20_000, 4, 80_000, 4),                              # a torus
    (5_003, 21, 50_000, 24),
    (5_003, 200, 50_000, 0),                             # a stride would cost twenty times the entries
    (9_000_000, 256, 792_000_000, 0),                    # 256 n > 2^31, three times the entries or not
    (8_388_604, 256, 8_388_604 * 88, 0),                 # just too many with the tail
    (8_388_540, 252, 8_388_540 * 88, 252),
    (1, 0, 0, 0),
])
def test_stride(ask, n, maxdeg, padded, stride):
    got, entries, fit = ask("s", n, maxdeg, padded)
    assert got == stride
    assert fit and 0 < entries <= INT32_MAX
    if stride:  # the last quad's reads stay inside
        assert entries >= stride * ((n + 3) // 4 * 4 - 1) + 16


def test_rows_that_do_not_fit(ask):
    assert ask("s", 8_400_000, 256, INT32_MAX - 16)[2] == 1
    assert ask("s", 8_400_000, 256, INT32_MAX - 15)[2] == 0
    # 253 entries a row: below 2^31 in the graph, above it padded
    assert ask("o", 8_400_000, 253, 1)[0] == 0
    assert ask("o", 1_000, 7, 7_000) == [3, 0, 8_000]
    assert ask("o", 1_000, 257, 1)[0] == 0


BITS, GATHERED, OTHERS = 0, 1, 2


@pytest.mark.parametrize("n,average,longest,tiles,form", [
    (3000, 4, 128, 1, BITS),          # long rows begin above 128 entries ..
    (3000, 4, 129, 1, OTHERS),
    (3000, 16, 128, 1, BITS),
    (3000, 20, 160, 64, BITS),        # .. and above 8 times the average
    (20000, 20, 161, 4, GATHERED),
    (3000, 8, 256, 1, OTHERS),
    (3000, 8, 256, 4, OTHERS),        # 768,000 spins
    (3000, 8, 256, 6, GATHERED),      # 1,152,000
    (3000, 8, 256, 87, GATHERED),     # 16,704,000
    (3000, 8, 256, 88, BITS),         # 16,896,000
    (20000, 8, 256, 2, OTHERS),
    (20000, 8, 256, 3, GATHERED),
    (8000, 20, 256, 2, BITS),         # 1,024,000
    (9000, 20, 256, 2, OTHERS),
    (9000, 20, 256, 3, BITS),
    (20000, 20, 256, 4, GATHERED),    # 5,120,000
])
def test_form_of_long_rows(ask, n, average, longest, tiles, form):
    got = ask("f", n, average * n, longest, tiles)
    # one or two rows above 64: never gathered without their fields kept
    assert got == [OTHERS if form == GATHERED else form, form]


@pytest.mark.parametrize("stride", [0, 1])
@pytest.mark.parametrize("both", [0, 1])
@pytest.mark.parametrize("n,m", [(1, 0), (2, 1), (5, 10), (41, 60), (64, 900)])
def test_row_entries(ask, n, m, both, stride):
    """Every row entry by entry: higher neighbours, lower ones, the zero mask."""
    rng = np.random.default_rng(n + both)
    pairs = {}
    while len(pairs) < m:
        u, v = sorted(int(x) for x in rng.integers(0, n, 2))
        if u != v:
            pairs[u, v] = 5 if not both or rng.random() < 0.5 else -5
    rows = [[] for _ in range(n)]
    for (u, v), w in pairs.items():
        rows[u].append((v, w))
        rows[v].append((u, w))
    for r in rows:
        rng.shuffle(r)
    ptr = np.concatenate([[0], np.cumsum([len(r) for r in rows])])
    flat = [(int(c), int(w)) for r in rows for c, w in r]
    out = ask("r", n, 2 * m, both, stride, *ptr, *(c for c, _ in flat), *(w for _, w in flat))
    np4, longest = (n + 3) // 4 * 4, max(len(r) for r in rows)
    step, size, out = out[0], out[1], out[2:]
    assert step == (stride and (longest + 3) // 4 * 4) and size == 4 * np4
    brows, ent = out[:size], out[size:]
    end = 0
    for v in range(np4):
        first, last = brows[2 * v], brows[2 * v + 1]
        if v >= n:
            assert first == last
            continue
        assert first == (v * step if step else end) and (last - first) % 4 == 0
        end = last
        want = [8 * (c + (np4 + 1 if both and w < 0 else 0)) for c, w in ([] if n == 1 else rows[v]) if c > v]
        below = [8 * (c + (np4 + 1 if both and w < 0 else 0)) for c, w in ([] if n == 1 else rows[v]) if c < v]
        deg = len(want) + len(below)
        assert sorted(ent[first:first + len(want)]) == sorted(want)
        assert sorted(ent[first + len(want):first + deg]) == sorted(below)
        assert set(ent[first + deg:last]) <= {8 * np4} and last - first - deg < 4
        assert brows[2 * np4 + v] == 4 * (longest - deg) and brows[3 * np4 + v] == len(want)
    assert len(ent) >= (np4 * step if step else end) + 16
    assert set(ent[end:]) == {8 * np4}
