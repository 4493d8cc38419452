"""Host arithmetic of csrc/splits.hpp: how the contraction of the weight-gradient products is cut, compiled by
the host compiler (no GPU)."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROGRAM = r'''
#include "splits.hpp"
#include <cstdio>
#include <cstdlib>
int main(int, char **v) {
  const int tiles = atoi(v[1]);
  const long long weights = atoll(v[2]), row_bytes = atoll(v[3]);
  for (int alone = 0; alone < 2; ++alone)
    for (long long M = 1; M <= 40000; M += M < 200 ? 1 : 61) {
      long long per = 0;
      const int n = snn::choose_splits(M, tiles, weights, row_bytes, &per, alone == 0);
      printf("%d %lld %d %lld\n", alone, M, n, per);
    }
}
'''


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    d = tmp_path_factory.mktemp("splits")
    (d / "main.cpp").write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++17", f"-I{ROOT}/paper_2402_18994_amd/csrc", "-o", str(d / "main"), str(d / "main.cpp")], check=True)
    return str(d / "main")


# one product of 100 x 16, 128 x 128 and 700 x 128, and the networks 100-64-10, 700-128-128-20, 700-256-256-20
@pytest.mark.parametrize("tiles,weights,row_bytes", [(1, 1600, 164), (1, 16384, 640), (6, 89600, 1212), (2, 7040, 460),
                                                     (8, 108544, 2060), (18, 249856, 3340)])
def test_splits_cover_the_rows_and_their_time_has_no_jump(program, tiles, weights, row_bytes):
    """Every row belongs to one split of a whole number of 64 rows, none of them empty; and where the chip is
    not full, the time of the longest split and of the partial sums (10 ns a row, 1.25 ps a partial sum) is within
    a third of the best count's, or 1 us of it: a count that falls to half from one length to the
    next, or does not know the partial sums, is not."""
    out = subprocess.run([program, str(tiles), str(weights), str(row_bytes)], check=True, capture_output=True, text=True).stdout
    rows = [tuple(map(int, line.split())) for line in out.splitlines()]
    assert len(rows) > 1000
    for alone, M, n, per in rows:
        assert per % 64 == 0 and n >= 1 and (n - 1) * per < M <= n * per, (M, n, per)
        if alone or M > 8192:
            continue

        def time(count):
            return 1e-2 * min(M, (-(-M // count) + 63) // 64 * 64) + 1.25e-6 * weights * count
        best = min(time(c) for c in (1, 2, 4, 8, 16, 32, 64) if c * tiles <= 256 or c == 1)
        assert time(n) <= max(4 / 3 * best, best + 1.0), (M, n, per)
