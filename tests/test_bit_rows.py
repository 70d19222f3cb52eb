"""Host arithmetic of the bit-packed sweeps' rows (csrc/bit_rows.hpp), built
with the host compiler: kernels and row bounds count entries in 32 bits, so
graphs whose rows would need more of them, with a stride or at all, are told
apart from those that fit."""
import os
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2606_25203_amd", "csrc")
INT32_MAX = 2**31 - 1

PROGRAM = r"""
#include "bit_rows.hpp"
#include <stdio.h>
#include <vector>
int main() {
  char what;
  long long a, b, c;
  while (scanf(" %c %lld %lld %lld", &what, &a, &b, &c) == 4) {
    if (what == 's') {  // stride of n rows, and the entries with it
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

    def run(what, a, b, c):
        out = subprocess.run([exe], input=f"{what} {a} {b} {c}\n", capture_output=True, text=True, check=True).stdout
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
