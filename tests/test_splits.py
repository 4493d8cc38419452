"""Host arithmetic of csrc/splits.hpp: how the contraction of the weight-gradient products is cut, compiled by
the host compiler (no GPU)."""
import os
import subprocess

import pytest

from tests.helpers import weight_gradient_form

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


# rows, sizes, recurrent layers, tiles of 256 x 128, their splits: where both kinds were timed, the faster one
TALL = [(65536, (700, 512, 512, 20), (), True, 11), (10000, (700, 512, 512, 20), (), False, 11),
        (65536, (700, 256, 256, 20), (), True, 28), (32768, (700, 256, 256, 20), (), False, 27),
        (65536, (300, 1024, 20), (), True, 12), (32768, (300, 1024, 20), (), False, 12),
        (57344, (700, 512, 20), (), True, 18), (40960, (700, 512, 20), (), False, 18),
        (131072, (700, 1024, 1024, 20), (), True, 9), (65536, (700, 2048, 2048, 2048, 20), (1, 0, 0), True, 4),
        (32768, (700, 128, 128, 20), (), False, 47), (3503, (398, 1911, 1911, 1911, 10), (), False, 2),
        (11235, (700, 1664, 1664, 10), (), True, 3)]


@pytest.mark.parametrize("M,sizes,recurrent,tall,splits", TALL, ids=["%d-rows-%s" % (t[0], "-".join(map(str, t[1]))) for t in TALL])
def test_which_weight_gradients_run_on_tall_tiles(M, sizes, recurrent, tall, splits):
    """The form, and the splits with the workgroups that are launched: every product has tiles of 256 x 128, also the
    narrow ones.  Every row belongs to one split, none of them is empty."""
    rec = tuple(recurrent) + (0,) * (len(sizes) - 2 - len(recurrent))
    got_tall, n, per, slots = weight_gradient_form(M, sizes, rec)
    assert (got_tall, n) == (tall, splits)
    assert per % 64 == 0 and (n - 1) * per < M <= n * per
    products = [(a, b) for a, b in zip(sizes, sizes[1:]) if not (b <= 32 and a > 128 and -(-a // 128) * M >= 3 << 18)]
    products += [(b, b) for b, r in zip(sizes[1:], rec) if r]
    assert slots == sum(-(-(-(-a // 256) * -(-b // 128) * n) // 8) for a, b in products)
