#!/usr/bin/env python3
"""Benchmark: training samples/s (forward + backward BPTT + SGD step) of the 700-128-128-20
LIF network at T=128, B=256 on one MI355X, with a roofline line for the dominant kernel, every
launch of the step against its own roof, and the CPU oracle timed beside it.

    python bench.py [--gpus 1] [--steps K] [--warmup W] [--workload shd_ff128] [--no-cpu]

Prints ONE JSON line on stdout; diagnostics go to stderr.

Order of the run: warm-up; the timed region (K steps, nothing bracketed: `value`); then, outside
it, K more steps with the dominant kernel bracketed by HIP events on the library's stream
(`roofline`), a few steps per kernel class and layer (`kernels`), forward + backward without the
optimiser step (`forward_backward_only`), the same shape with fp32 products (`fp32_products`), and
the oracle on the host cores (`cpu_baseline`).
"""
import argparse
import json
import os
import sys
import time

ROOT = os.path.dirname(os.path.abspath(__file__))
if ROOT not in sys.path:
    sys.path.insert(0, ROOT)

HBM_PEAK_GBS = 8000.0          # MI355X HBM3E
MFMA_BF16_PEAK_TFLOPS = 2500.0  # dense bf16 MFMA

# HBM bytes per launch of the dominant kernel as counted by rocprofv3 --pmc (FETCH_SIZE run, then
# WRITE_SIZE run; KiB per dispatch, each scaled by what the same counter reads for the 256 MiB
# device copy this script issues first: FETCH_SIZE reads half the bytes of that copy, WRITE_SIZE
# all of them).  Not measured by this run: the figure is the one in the named summary, which the
# same command produced under the profiler; --traffic replaces it.
PROFILED_TRAFFIC = {           # (workload, kernel, input packed along time)
    ("shd_ff128", "lif_forward", False): ((15841.0 * 2.0 + 50256.0) * 1024.0, "profiles/train_step_shd_ff128.txt"),
    ("shd_ff128", "lif_forward", True): ((4523.0 * 2.0 + 50256.0) * 1024.0, "profiles/train_step_shd_ff128.txt"),
}


def pad8(n):
    return (n + 7) // 8 * 8


def adaptive(wl, layer):
    return bool(wl.adapt_step) and wl.adapt_step[layer - 1] > 0


def runs_whole(wl, l):
    """Whether text layer l runs product and scan as one forward launch (the library's default rule)."""
    L = len(wl.sizes) - 1
    if not (1 <= l < L) or wl.recurrent[l - 1]:
        return False
    n = pad8(wl.sizes[l])
    k = wl.sizes[0] if l == 1 and wl.sizes[0] % 4 == 0 else pad8(wl.sizes[l - 1])
    if n > 1024 or k > 1024:
        return False
    T, B, bf, fan_in = wl.T, wl.B, wl.precision == "bf16", wl.sizes[l - 1]
    blocks = -(-T // 128)
    rounds = blocks * -(-fan_in // 64)
    if adaptive(wl, l):
        groups = B * -(-n // 64)
        if T > 256 or wl.theta + wl.adapt_step[l - 1] * T > 2.0 ** 26:
            return False
        if 128 < T < (176 if groups > 1536 else 160 if groups < 256 else 0):
            return False
        if T > 128 and bf and groups > 1536 and n > 768 and n % 64:
            return False
        if fan_in <= 256 and not (T > 40 and (T <= 64 or T * 5 >= blocks * 128 * 4)):
            return False
        return bf or rounds <= 16 or B >= 64
    company = narrow_in_company(wl, l)
    per = (64 if company <= 64 else 128) if company else 64 if -(-n // 64) * 64 < -(-n // 128) * 128 else 128
    groups = B * -(-n // per)
    if bf:
        if T <= (384 if company or per == 64 else 256) or (company and per == 64) or (T <= 512 and rounds <= 16):
            return True
        if top_scan_forms_currents(wl, L - 1) and (l == L - 1 or l == L - 2 and company and narrow_in_company(wl, L - 1)):
            return True

        def full(i):
            return 1 <= i < L and pad8(wl.sizes[i]) == 128 and narrow_in_company(wl, i)
        if full(l) and (full(l - 1) or full(l + 1)):
            return T <= 512 or groups >= (32 if T <= 1024 else 80)
        return groups >= (32 if rounds <= 16 else 64 if rounds <= 32 or T <= 512 else 80 if T <= 1024 else 128)
    if T <= 128 or (T <= 256 and rounds <= (16 if company else 8)):
        return True
    if rounds <= 16:
        if (per == 64 or T <= 384) if company else (per == 64 and T <= 512):
            return True
        return groups >= (32 if company and T <= 512 else 64 if T <= 768 else 128)
    return groups >= (192 if rounds > 64 else 64 if company and (per == 64 or T <= 768) else 128)


def narrow_in_company(wl, l):
    """For a layer of at most 128 neurons whose launch holds the readout or a second such layer too: the widest of the
    layers that can be in it; else 0."""
    L = len(wl.sizes) - 1

    def narrow(i):
        is_narrow = 1 <= i < L and pad8(wl.sizes[i]) <= 128 and not wl.recurrent[i - 1] and not adaptive(wl, i)
        return pad8(wl.sizes[i]) if is_narrow else 0
    if not narrow(l) or not ((l == L - 1 and pad8(wl.sizes[L]) <= 32) or narrow(l - 1) or narrow(l + 1)):
        return 0
    return max(narrow(l), narrow(l - 1), narrow(l + 1))


def top_scan_forms_currents(wl, layer):
    """Whether the scan of the last spiking layer, where it is a launch of its own, forms the readout's currents."""
    L = len(wl.sizes) - 1
    return (layer == L - 1 and wl.precision == "bf16" and not wl.recurrent[layer - 1] and not adaptive(wl, layer)
            and pad8(wl.sizes[layer]) in (64, 128, 256) and pad8(wl.sizes[L]) <= 32)


def forward_wide(wl, layer):
    """Whether text layer `layer` runs on the kernel for wide layers (two samples and 128 neurons to a workgroup): more
    than 128 neurons, rounded weights, where there are workgroups enough, or by the library's estimate (us) against product
    and scan apart."""
    L = len(wl.sizes) - 1
    if not (1 <= layer < L) or wl.precision != "bf16" or wl.recurrent[layer - 1] or adaptive(wl, layer) or pad8(wl.sizes[layer]) <= 128:
        return False
    n, fan_in, rows = pad8(wl.sizes[layer]), wl.sizes[layer - 1], wl.T * wl.B
    parts = -(-n // 128)
    if runs_whole(wl, layer):
        return wl.T > 64 and -(-n // 64) * 64 == parts * 128 and wl.B * parts >= 768
    if top_scan_forms_currents(wl, layer):
        return False
    rounds = max(1, (wl.B + 1) // 2 * parts / 256)
    one = 4 + -(-wl.T // 128) * rounds * (10.5 + 0.5 * -(-fan_in // 64))
    product = 3 + (1.5e-9 if rows * n * 4 >= 128 << 20 else 2.5e-9) * rows * n * fan_in + 4 * rows * n / 5e6
    return 1.1 * one < product + max(0.043 * wl.T + 2, 2 + 9 * rows * n / 6e6)


def forward_chain(wl, layer):
    """The spiking layers that the forward launch starting at text layer `layer` covers, and whether it
    runs the readout too; ([], False) if that layer runs as separate product and scan launches."""
    L = len(wl.sizes) - 1
    if not runs_whole(wl, layer):
        return [], False

    def joins(l):
        return l < L and pad8(wl.sizes[l]) <= 128 and not adaptive(wl, l)

    def pairs(l):
        return joins(l) and joins(l + 1) and runs_whole(wl, l) and runs_whole(wl, l + 1)

    def like(l):                     # workgroups of the same width
        return (pad8(wl.sizes[l]) > 64) == (pad8(wl.sizes[l + 1]) > 64)
    chain = [layer]
    if pairs(layer) and (like(layer) or not (pairs(layer + 1) and like(layer + 1))):
        chain.append(layer + 1)
    top = chain[-1]
    return chain, top == L - 1 and joins(top) and pad8(wl.sizes[L]) <= 32


def forward_launch(wl, layer):
    """forward_chain, with the layers that run on the kernel for wide layers."""
    return ([layer], False) if forward_wide(wl, layer) else forward_chain(wl, layer)


def reverse_wide(wl, layer):
    """Whether the reverse pass of text layer `layer`, feed-forward on rounded weights and below more than 128 columns or
    adaptive, runs as one launch: the library's estimate of its time (us) against that of product and scan."""
    if not (1 <= layer < len(wl.sizes) - 1):
        return False
    n, above, rows = pad8(wl.sizes[layer]), pad8(wl.sizes[layer + 1]), wl.T * wl.B
    a = adaptive(wl, layer)
    if wl.precision != "bf16" or wl.recurrent[layer - 1] or (above <= 128 and not a):
        return False
    groups = wl.B * -(-n // 256)
    rounds = -(-groups // 256) if groups <= 512 else groups / 256
    one = 4 + -(-wl.T // 128) * rounds * ((12 if a else 9) + 0.62 * -(-above // 32))
    product = 3 + 2.4e-9 * rows * n * above + 4 * rows * (n + above) / 5e6
    scan = max(0.062 * wl.T + 2, 2 + 16 * rows * n / 5.2e6) if a else max(0.048 * wl.T + 1, 2 + 12 * rows * n / 5.2e6)
    return 1.15 * one < product + scan + 2


def reverse_forms_ds(wl, layer):
    """Whether the reverse launch of text layer `layer` forms dS from the current gradients above itself
    (feed-forward, at most 128 padded columns above; up to 1024 neurons, or any multiple of 64 on rounded weights).
    Below wider layers, and with adaptive thresholds: reverse_wide."""
    L = len(wl.sizes) - 1
    if not (1 <= layer < L) or wl.recurrent[layer - 1] or adaptive(wl, layer) or pad8(wl.sizes[layer + 1]) > 128:
        return False
    n, bf = pad8(wl.sizes[layer]), wl.precision == "bf16"
    least = 32 if not bf and pad8(wl.sizes[layer + 1]) > 64 and wl.T > 256 else 1
    return (bf and n % 64 == 0) or (n <= 1024 and wl.B >= least)


def recurrent_pair(wl, layer):
    """Whether text layer `layer` and the one above it share a launch per direction: recurrent, rounded weights,
    at most 192 neurons each and sixteen wavefronts with those of the product between them, up to 2048 samples;
    taken from the bottom up."""
    L = len(wl.sizes) - 1
    if not (1 <= layer < L - 1) or wl.precision != "bf16" or wl.B > 2048 or not (wl.recurrent[layer - 1] and wl.recurrent[layer]):
        return False
    n = [pad8(v) for v in wl.sizes[layer:layer + 2]]
    waves = [-(-v // 32) for v in n]
    return max(n) <= 192 and sum(waves) + max(waves) <= 16 and not recurrent_pair(wl, layer - 1)


def algorithmic_bytes(wl, kernel, layer, packed=False):
    """HBM bytes one launch of `kernel` for text layer `layer` has to move (compulsory traffic
    of its operands and results, each touched once), in the formats this build stores; `packed`:
    the input raster is read as eight steps per byte."""
    M = wl.T * wl.B
    # rows of the raster as the launches of layer 1 read it (they read the bits themselves where layer 1
    # runs as one launch and, for the weight gradient, the batch is a multiple of 8; else a pre-pass unpacks)
    direct = packed and wl.sizes[0] % 4 == 0 and runs_whole(wl, 1) and (kernel != "weight_grad" or wl.B % 8 == 0)
    x_rows = (wl.T + 7) // 8 * wl.B if direct else M
    bf = wl.precision == "bf16"
    di = 4                           # current gradients are 4 bytes in memory in both modes
    planes = 1 if bf else 3
    L = len(wl.sizes) - 1
    if kernel == "weight_grad" and layer == 0:   # the merged launch: every layer's spikes below, dI and dW (+ dR)
        return sum(algorithmic_bytes(wl, kernel, l, packed) for l in range(1, L + 1))
    n_in, n_out = wl.sizes[layer - 1], wl.sizes[layer]
    fused_rev = reverse_forms_ds(wl, layer) or reverse_wide(wl, layer)
    fused_fwd = top_scan_forms_currents(wl, layer)
    state = 4 if layer < L and adaptive(wl, layer) else 0        # the adaptation, beside V
    chain, with_readout = forward_launch(wl, layer)
    if kernel == "lif_forward" and chain:
        # the launch that starts at `layer`: spikes below (1 B) and W (2 B a plane) read; V (4) and S (1) written
        # per layer; with the readout its currents, its trace and its current gradients (4 B each)
        total = (x_rows if layer == 1 else M) * n_in
        for l in chain:
            total += planes * 2 * wl.sizes[l - 1] * wl.sizes[l] + M * wl.sizes[l] * (4 + 1 + state)
        if with_readout:
            total += planes * 2 * wl.sizes[chain[-1]] * wl.sizes[L] + 3 * M * pad8(wl.sizes[L]) * 4
        return total
    if kernel == "lif_forward":      # read I (4), write V (4) and S (1 byte) [+ the readout's currents]
        return M * n_out * (4 + 4 + 1 + state) + (M * pad8(wl.sizes[L]) * 4 if fused_fwd else 0)
    if kernel == "lif_reverse":      # read dS (4) [or the current gradients above] and V (4), write dI (4)
        above = pad8(wl.sizes[layer + 1]) if fused_rev else n_out
        return M * (above * 4 + n_out * (4 + di + state))
    if kernel == "current_gemm":     # read spikes (1 byte) and the weight planes, write I (4)
        return M * n_in + planes * 2 * n_in * n_out + M * n_out * 4
    if kernel == "weight_grad":      # read spikes and dI, write dW (recurrent: own spikes too, and dR)
        rec = layer < L and wl.recurrent[layer - 1]
        return (x_rows if layer == 1 else M) * n_in + M * n_out * di + n_in * n_out * 4 + (M * n_out + n_out * n_out * 4 if rec else 0)
    if kernel == "input_grad":       # read dI and the weight planes, write dS
        return M * n_out * di + planes * 2 * n_in * n_out + M * n_in * 4
    if kernel == "readout_forward":  # J read, Y and dJ written (4 B per padded class)
        return 3 * M * pad8(wl.sizes[L]) * 4
    if kernel == "readout_reverse":
        return M * pad8(wl.sizes[L]) * 4
    raise KeyError(kernel)


def method_flops(wl, kernel, layer):
    """Multiply-add flops of the method (one pass over the operands; a hi+lo or three-piece operand
    is still one product) that one launch of `kernel` for text layer `layer` contains."""
    M = wl.T * wl.B
    L = len(wl.sizes) - 1
    if kernel == "weight_grad" and layer == 0:
        return sum(method_flops(wl, kernel, l) for l in range(1, L + 1))
    n_in, n_out = wl.sizes[layer - 1], wl.sizes[layer]
    if kernel == "lif_forward":
        chain, with_readout = forward_launch(wl, layer)
        f = sum(2 * M * wl.sizes[l - 1] * wl.sizes[l] for l in chain)
        if with_readout:
            f += 2 * M * wl.sizes[chain[-1]] * wl.sizes[L]
        elif not chain and top_scan_forms_currents(wl, layer):
            f += 2 * M * n_out * wl.sizes[L]
        return f
    if kernel == "lif_reverse":
        return 2 * M * n_out * wl.sizes[layer + 1] if reverse_forms_ds(wl, layer) or reverse_wide(wl, layer) else 0
    if kernel in ("current_gemm", "input_grad"):
        return 2 * M * n_in * n_out
    if kernel == "weight_grad":
        rec = layer < L and wl.recurrent[layer - 1]
        return 2 * M * n_in * n_out + (2 * M * n_out * n_out if rec else 0)
    if kernel in ("rlif_forward", "rlif_reverse"):       # a pair: both layers' own products and the one between them
        up = wl.sizes[layer + 1] if recurrent_pair(wl, layer) else 0
        return 2 * M * (n_out * n_out + n_out * up + up * up)
    return 0


def gemm_flops(wl):
    M = wl.T * wl.B
    f = 0
    for l in range(1, len(wl.sizes)):
        k, n = wl.sizes[l - 1], wl.sizes[l]
        f += 2 * M * k * n            # current product
        f += 2 * M * k * n            # weight gradient
        if l > 1:
            f += 2 * M * k * n        # input gradient
    for l, rec in enumerate(wl.recurrent):
        if rec:
            n = wl.sizes[l + 1]
            f += 3 * 2 * M * n * n    # S R, g R^T, dR
    return f


def roof_entry(us, nbytes, flops):
    """One launch against its own roof: min(MFMA peak, arithmetic intensity x HBM peak)."""
    e = {"us": round(us, 2)}
    if nbytes:
        e["algorithmic_bytes"] = int(nbytes)
        e["gb_per_s"] = round(nbytes / us / 1e3, 1)
        e["hbm_frac"] = round(nbytes / us / 1e3 / HBM_PEAK_GBS, 3)
    if flops:
        e["method_flops"] = int(flops)
        e["tflop_per_s"] = round(flops / us / 1e6, 1)
        e["mfma_frac"] = round(flops / us / 1e6 / MFMA_BF16_PEAK_TFLOPS, 3)
    if nbytes or flops:
        floor_us = max(nbytes / (HBM_PEAK_GBS * 1e3), flops / (MFMA_BF16_PEAK_TFLOPS * 1e6))
        e["bound"] = "mfma" if flops / (MFMA_BF16_PEAK_TFLOPS * 1e6) > nbytes / (HBM_PEAK_GBS * 1e3) else "hbm"
        e["roof_frac"] = round(floor_us / us, 3)
    return e


def cpu_baseline(wl, inp, budget_s=12.0):
    """The oracle as it stands, whole training steps on the host cores."""
    import numpy as np
    from oracle import snn_oracle as O
    from tests.helpers import net_of
    blas = None
    try:
        from threadpoolctl import threadpool_info
        blas = max([p.get("num_threads", 1) for p in threadpool_info()] or [1])
    except Exception:
        pass
    net = net_of(wl)
    W, R = [w.astype(np.float64) for w in inp.W], inp.R
    O.train_step(net, inp.X, W, R, inp.labels, 0.01)          # warm-up
    t0 = time.perf_counter()
    n = 0
    while True:
        _, _, W, R = O.train_step(net, inp.X, W, R, inp.labels, 0.01)
        n += 1
        dt = time.perf_counter() - t0
        if dt >= budget_s or n >= 50:
            break
    return {"value": wl.B * n / dt, "unit": "samples/s", "cores": int(os.cpu_count() or 1),
            "blas_threads": blas, "kind": "oracle",
            "sample": f"{n} full training steps (forward+backward+SGD) of the same batch, "
                      f"T={wl.T} B={wl.B}, NumPy float64, {dt:.1f} s"}


def main():
    ap = argparse.ArgumentParser()
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=200)
    ap.add_argument("--warmup", type=int, default=20)
    ap.add_argument("--workload", default="shd_ff128")
    ap.add_argument("--dominant", default=None,
                    help="kernel:layer bracketed for the roofline line (layer 0 = every layer)")
    ap.add_argument("--traffic", type=float, default=None,
                    help="HBM bytes per launch of the dominant kernel from rocprofv3 --pmc runs of this command")
    ap.add_argument("--packed", action="store_true",
                    help="feed the raster packed along time (eight spikes per byte) through snn_forward_packed")
    ap.add_argument("--option", action="append", default=[], metavar="NAME=VALUE",
                    help="kernel-selection option of the context (binding.OPTIONS), repeatable")
    ap.add_argument("--no-cpu", action="store_true")
    ap.add_argument("--no-extras", action="store_true",
                    help="skip the per-launch table and the fp32-products run (profiler runs)")
    args = ap.parse_args()
    if args.gpus != 1:
        print("bench.py: this build runs on ONE GPU only; --gpus must be 1", file=sys.stderr)
        sys.exit(2)

    import numpy as np
    import torch
    import workloads
    from paper_2402_18994_amd.binding import from_workload, CALIBRATE_US

    if not torch.cuda.is_available():
        print("bench.py: no HIP device; there is no CPU path to time", file=sys.stderr)
        sys.exit(3)
    wl = workloads.CONFIGS[args.workload]
    inp = workloads.generate(wl)
    dev = torch.device("cuda:0")
    options = {k: int(v) for k, v in (o.split("=", 1) for o in args.option)}
    snn = from_workload(wl, inp, device="cuda:0", options=options or None)
    x = torch.from_numpy(inp.X).to(dev)
    y = torch.from_numpy(inp.labels).to(dev)
    lr = 1e-3
    L = len(wl.sizes) - 1

    if args.packed:
        xp = torch.from_numpy(np.packbits(inp.X, axis=0)).to(dev)

    def step(net=snn):
        if args.packed:
            net.forward_packed(xp, y, want_loss=False)
        else:
            net.forward(x, y, want_loss=False)
        net.backward()
        net.sgd_step(lr)

    # A plain device copy of known size: the reference the FETCH_SIZE / WRITE_SIZE counters of a
    # rocprofv3 --pmc run are scaled by (256 MiB read, 256 MiB written; the source is pushed out
    # of the caches first by writing 512 MiB elsewhere).
    cal_src = torch.zeros(256 << 20, dtype=torch.uint8, device=dev)
    cal_dst = torch.empty_like(cal_src)
    torch.empty(512 << 20, dtype=torch.uint8, device=dev).zero_()
    cal_dst.copy_(cal_src)
    del cal_src, cal_dst
    torch.cuda.synchronize()
    torch.cuda.empty_cache()

    for _ in range(args.warmup):
        step()
    torch.cuda.synchronize()

    # ------------------------------------------------------------ the timed region: nothing bracketed
    snn.profile_select("none", 0)
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    for _ in range(args.steps):
        step()
    torch.cuda.synchronize()
    dt = time.perf_counter() - t0
    ms_per_step = dt / args.steps * 1e3
    value = wl.B * args.steps / dt

    # ------------------------------------------------------------ kernel durations, outside the timed region
    # An event pair brackets a launch on the library's stream.  What the pair adds to the launch it
    # brackets is measured in this run: the library brackets a one-wavefront kernel that waits
    # CALIBRATE_US on the device clock, once per step, in the middle of the backward pass; the excess
    # over CALIBRATE_US is subtracted from every bracketed launch.  Durations are therefore on the
    # device clock's scale: the calibration kernel counts as exactly its wait (rocprofv3 reports
    # about 1 us more for it, the start and end of a dispatch, which its durations include).
    # (A bracket around nothing costs more than it adds to a launch, so it is only reported.)
    def bracketed(name, layer, n):
        snn.profile_select(name, layer)
        for _ in range(n):
            step()
        ms, launches = snn.profile_read()
        return ms * 1e3, launches                      # microseconds in all, launches in all

    us, n = bracketed("event_pair", 0, 50)
    empty_pair_us = us / max(1, n)
    us, n = bracketed("calibrate", 0, 50)
    cal_raw_us = us / max(1, n)
    pair_us = cal_raw_us - CALIBRATE_US                 # what a bracket adds to the launch inside it

    if args.dominant is None:
        # the launch with the largest share of the step: where the forward pass of all spiking layers and the
        # readout is one launch, that one; else the merged weight-gradient launch
        chain, with_readout = forward_launch(wl, 1)
        args.dominant = "lif_forward:1" if with_readout and len(chain) == L - 1 else "weight_grad:0"
    kname, klayer = args.dominant.split(":")
    klayer = int(klayer)
    blayer = klayer if (klayer or kname == "weight_grad") else 1
    k_us, k_n = bracketed(kname, klayer, args.steps)   # the same number of steps as the timed region
    k_raw_us = k_us / max(1, k_n)
    k_avg_us = max(k_raw_us - pair_us, 1e-3)
    abytes = algorithmic_bytes(wl, kname, blayer, args.packed)
    achieved = abytes / k_avg_us / 1e3 if k_n else 0.0

    kernels = []
    if not args.no_extras:
        todo = [("lif_forward", l) for l in range(1, L)] + [("rlif_forward", l) for l in range(1, L)]
        todo += [("current_gemm", l) for l in range(1, L + 1)] + [("readout_forward", L), ("readout_reverse", L)]
        todo += [("lif_reverse", l) for l in range(L - 1, 0, -1)] + [("rlif_reverse", l) for l in range(L - 1, 0, -1)]
        todo += [("input_grad", l) for l in range(L, 1, -1)] + [("weight_grad", 0), ("grad_reduce", 0), ("sgd", 0)]
        reps = 10
        for name, layer in todo:
            us, n = bracketed(name, layer, reps)
            if not n:
                continue
            per_launch = us / n - pair_us
            nb = fl = 0
            try:
                nb = algorithmic_bytes(wl, name, layer if layer else 0, args.packed) if name not in ("rlif_forward", "rlif_reverse", "grad_reduce", "sgd") else 0
            except KeyError:
                nb = 0
            fl = method_flops(wl, name, layer)
            e = {"kernel": name, "layer": layer, "launches_per_step": n // reps}
            if n // reps > 1:                           # one launch per time step: no roof claimed (latency-bound)
                e["us"] = round(per_launch, 2)
                e["us_per_step_all_launches"] = round(per_launch * (n // reps), 1)
            else:
                e.update(roof_entry(max(per_launch, 1e-3), nb, fl))
            kernels.append(e)
    snn.profile_select("none", 0)

    # Forward + backward alone (the metric as BASELINE words it, without the optimiser step): the
    # backward pass then adds the weight gradients' partial sums itself instead of leaving them to
    # snn_sgd_step, so the gradients are complete when it returns.
    fwd_bwd = None
    if not args.no_extras:
        snn.set_option("defer_reduce", 0)
        nfb = max(20, args.steps // 2)

        def fb():
            if args.packed:
                snn.forward_packed(xp, y, want_loss=False)
            else:
                snn.forward(x, y, want_loss=False)
            snn.backward()
        for _ in range(5):
            fb()
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        for _ in range(nfb):
            fb()
        torch.cuda.synchronize()
        dfb = time.perf_counter() - t0
        fwd_bwd = {"value": wl.B * nfb / dfb, "unit": "samples/s", "ms_per_step": dfb / nfb * 1e3, "steps": nfb,
                   "what": "snn_forward + snn_backward, gradients reduced, no snn_sgd_step"}
        snn.set_option("defer_reduce", options.get("defer_reduce", 1))

    loss = snn.forward(x, y)
    spike_rate = [float(snn.get_tensor("spikes", l).mean()) for l in range(1, L)]
    snn.destroy()

    out = {
        "metric": "training samples/sec (fwd+bwd BPTT + SGD step), T=%d, B=%d" % (wl.T, wl.B),
        "value": value, "unit": "samples/s", "n_gpus": 1, "steps": args.steps, "warmup": args.warmup,
        "ms_per_step": ms_per_step, "higher_is_better": True, "scaling": "weak", "vs_baseline": None,
        "dtype": "bf16" if wl.precision == "bf16" else "f32", "data": "synthetic",
        "config": {"workload": f"{wl.name}: {'-'.join(map(str, wl.sizes))} LIF, T={wl.T}, B={wl.B}, "
                               f"recurrent={list(map(int, wl.recurrent))}, {wl.surrogate}({wl.slope:g}), "
                               f"bf16 products / fp32 state" + (", input packed along time" if args.packed else "")
                               if wl.precision == "bf16" else
                               f"{wl.name}: {'-'.join(map(str, wl.sizes))}, T={wl.T}, B={wl.B}, fp32",
                   "options": options, "final_loss": loss, "spike_rate": spike_rate,
                   "note": "weights N(0, 1/sqrt(fan_in)) as the configuration states them: the hidden layers are "
                           "almost silent; no kernel branches on a spike, so the time per step does not depend on it"},
        "roofline": {"bound": "hbm", "kernel": f"{kname}" + (f" layer {klayer}" if klayer else " (all layers)"),
                     "achieved": achieved, "peak": HBM_PEAK_GBS, "unit": "GB/s", "frac": achieved / HBM_PEAK_GBS,
                     "traffic": None, "traffic_source": None,
                     "algorithmic_bytes_per_launch": abytes,
                     "avg_launch_us": k_avg_us, "avg_launch_us_with_events": k_raw_us,
                     "event_pair_overhead_us": pair_us, "launches": k_n,
                     "calibration_kernel_with_events_us": cal_raw_us, "calibration_kernel_waits_us": CALIBRATE_US,
                     "empty_event_pair_us": empty_pair_us,
                     "timed": "HIP events on the library's stream, %d steps after the timed region" % args.steps},
        "gemm_tflops_whole_step": gemm_flops(wl) / (dt / args.steps) / 1e12,
        "kernels": kernels,
    }
    if fwd_bwd:
        out["forward_backward_only"] = fwd_bwd
    if args.traffic is not None:
        out["roofline"]["traffic"] = args.traffic
        out["roofline"]["traffic_source"] = "--traffic"
    elif (wl.name, kname, args.packed) in PROFILED_TRAFFIC and not options:
        out["roofline"]["traffic"], out["roofline"]["traffic_source"] = PROFILED_TRAFFIC[(wl.name, kname, args.packed)]

    if not args.no_extras and wl.precision == "bf16":
        # The same shape with fp32 products (the arithmetic of the paper's timing runs, Section 3.1): every
        # real operand enters the MFMA units as three bfloat16 pieces.
        wl32 = wl.scaled(precision="fp32")
        snn32 = from_workload(wl32, inp, device="cuda:0")
        n32 = max(5, args.steps // 4)
        for _ in range(3):
            step(snn32)
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        for _ in range(n32):
            step(snn32)
        torch.cuda.synchronize()
        d32 = time.perf_counter() - t0
        out["fp32_products"] = {"value": wl.B * n32 / d32, "unit": "samples/s", "ms_per_step": d32 / n32 * 1e3,
                                "steps": n32, "final_loss": snn32.forward(x, y)}
        snn32.destroy()

    if not args.no_cpu:
        out["cpu_baseline"] = cpu_baseline(wl, inp)
    print(json.dumps(out))


if __name__ == "__main__":
    main()
