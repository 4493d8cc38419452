"""Host arithmetic of csrc/wide_rules.hpp, which says what layers run on the kernels for wide layers, compiled by the host
compiler (no GPU), against bench.py's account of the same."""
import random
import subprocess

import pytest

import bench
import workloads
from tests.helpers import host_program

PROGRAM = r'''
#include "wide_rules.hpp"
#include <cstdio>
int main() {                     // per line: T B ld fan_in columns adaptive one_launch top_scan streams
  int T, B, ld, fan_in, columns, adaptive, one_launch, top_scan, streams;
  while (scanf("%d %d %d %d %d %d %d %d %d", &T, &B, &ld, &fan_in, &columns, &adaptive, &one_launch, &top_scan, &streams) == 9)
    printf("%d %d\n", (int)snn::forward_wide_pays(T, B, ld, fan_in, one_launch, top_scan, streams),
           (int)snn::reverse_wide_pays(T, B, ld, columns, adaptive));
}
'''


def test_bench_accounts_for_wide_layers_as_the_library_decides():
    rng = random.Random(5)
    cases, asked = [], []
    for _ in range(6000):
        T, B = int(2 ** rng.uniform(4, 9.5)), int(2 ** rng.uniform(2, 9))
        sizes = (rng.choice((700, rng.randrange(40, 1000))),) + tuple(int(2 ** rng.uniform(6, 11)) for _ in range(rng.choice((1, 2, 2)))) + (rng.choice((10, 20, 150)),)
        L, adaptive = len(sizes) - 1, rng.random() < 0.3
        kw = dict(adapt_decay=(0.9,) * (L - 1), adapt_step=(0.2,) * (L - 1)) if adaptive else {}
        wl = workloads.Workload(name="rule", index=0, T=T, B=B, sizes=sizes, recurrent=(False,) * (L - 1), beta=(0.9,) * L, theta=1.0,
                                surrogate="superspike", slope=10.0, precision="bf16", rate_lo=0.1, rate_hi=0.2, **kw)
        l = rng.randrange(1, L)
        cases.append((wl, l, adaptive))
        n = bench.pad8(sizes[l])
        asked.append("%d %d %d %d %d %d %d %d %d" % (T, B, n, sizes[l - 1], bench.pad8(sizes[l + 1]), adaptive, bench.runs_whole(wl, l),
                                                     bench.top_scan_forms_currents(wl, l), T * B * n * 4 >= 128 << 20))
    out = subprocess.run([host_program(PROGRAM)], input="\n".join(asked), check=True, capture_output=True, text=True).stdout
    seen = set()
    for (wl, l, adaptive), line in zip(cases, out.splitlines()):
        forward, reverse = (v == "1" for v in line.split())
        n, above = bench.pad8(wl.sizes[l]), bench.pad8(wl.sizes[l + 1])
        assert bench.forward_wide(wl, l) == (forward and n > 128 and not adaptive), (wl, l)
        assert bench.reverse_wide(wl, l) == (reverse and (above > 128 or adaptive)), (wl, l)
        seen.add((forward, reverse, adaptive))
    assert len(seen) == 8


@pytest.mark.parametrize("layer_forward,max_neurons,neurons,time_split", [(4, 1024, 128, 0), (3, 1024, 128, 0), (4, 960, 128, 0), (4, 1024, 64, 0),
                                                                          (4, 1024, 128, 1)])
def test_options_that_ask_for_another_forward_kernel_are_heard(layer_forward, max_neurons, neurons, time_split):
    program = host_program('#include "wide_rules.hpp"\n#include <cstdio>\n#include <cstdlib>\nint main(int, char **v) {'
                           ' printf("%d", (int)snn::forward_wide_allowed(atoi(v[1]), atoi(v[2]), atoi(v[3]), atoi(v[4]))); }')
    options = (layer_forward, max_neurons, neurons, time_split)
    out = subprocess.run([program] + list(map(str, options)), check=True, capture_output=True, text=True).stdout
    assert out == str(int(options == (4, 1024, 128, 0)))
