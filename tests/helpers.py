"""Shared test helpers: workload -> oracle Net conversion, tiny random nets."""
import functools
import os
import subprocess
import tempfile

import numpy as np

from oracle.snn_oracle import Net

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2402_18994_amd", "csrc")


@functools.lru_cache(None)
def host_program(text):
    """The path of a program that includes the library's host headers, built by the host compiler."""
    d = tempfile.mkdtemp(prefix="snn_host_")
    main = os.path.join(d, "main")
    with open(main + ".cpp", "w") as f:
        f.write(text)
    subprocess.run(["g++", "-std=c++17", "-I" + CSRC, "-o", main, main + ".cpp"], check=True)
    return main


WEIGHT_GRADIENT_FORM = r'''
#include "splits.hpp"
#include <cstdio>
#include <cstdlib>
int main(int argc, char **v) {   // M, then per layer its size and whether it is recurrent
  const long long M = atoll(v[1]);
  std::vector<int> sizes;
  std::vector<bool> recurrent;
  for (int i = 2; i < argc; i += 2) { sizes.push_back(atoi(v[i])); if (i > 2) recurrent.push_back(atoi(v[i + 1])); }
  const snn::WgradLaunch w = snn::wgrad_launch(M, (int)sizes.size() - 1, sizes.data(), recurrent, false);
  long long per = 0;
  const int splits = snn::choose_splits_tall(M, w, &per);
  printf("%d %d %lld %lld\n", (int)snn::wgrad_tall_pays(M, w), splits, per, snn::tall_slots(w, splits));
}
'''


def weight_gradient_form(M, sizes, recurrent):
    """The library's rules for the weight gradients of a network on rounded weights, M rows each: whether they run on tiles of
    256 x 128, and on those the splits of the launch, the rows of one and the workgroups of an XCD."""
    args = [str(M)]
    for n, r in zip(sizes, (0,) + tuple(recurrent) + (0,)):
        args += [str(n), str(int(r))]
    out = subprocess.run([host_program(WEIGHT_GRADIENT_FORM)] + args, check=True, capture_output=True, text=True).stdout
    tall, splits, per, slots = map(int, out.split())
    return bool(tall), splits, per, slots


def net_of(wl, gemm_round=None):
    rnd = gemm_round if gemm_round is not None else ("bf16" if wl.precision == "bf16" else "none")
    return Net(sizes=tuple(wl.sizes), recurrent=tuple(wl.recurrent), beta=tuple(wl.beta),
               theta=wl.theta, surrogate=wl.surrogate, slope=wl.slope, gemm_round=rnd,
               loss=getattr(wl, "loss", "max"), adapt_decay=getattr(wl, "adapt_decay", None),
               adapt_step=getattr(wl, "adapt_step", None))


def tiny_net(rng, sizes=(5, 4, 6, 3), recurrent=(False, True), T=7, B=2, surrogate="sigmoid",
             slope=3.0, beta=(0.9, 0.8, 0.85), theta=1.0, p=0.5, gain=1.5, gemm_round="none", loss="max",
             adapt_decay=None, adapt_step=None):
    net = Net(sizes=tuple(sizes), recurrent=tuple(recurrent), beta=tuple(beta), theta=theta,
              surrogate=surrogate, slope=slope, gemm_round=gemm_round, loss=loss,
              adapt_decay=adapt_decay, adapt_step=adapt_step)
    L = len(sizes) - 1
    X = (rng.random((T, B, sizes[0])) < p).astype(np.uint8)
    W = [rng.standard_normal((sizes[l], sizes[l + 1])) * gain / np.sqrt(sizes[l]) for l in range(L)]
    R = [rng.standard_normal((sizes[l + 1], sizes[l + 1])) * 0.5 / np.sqrt(sizes[l + 1])
         if recurrent[l] else None for l in range(L - 1)]
    labels = rng.integers(0, sizes[-1], size=B)
    return net, X, W, R, labels
