"""Host-side checks of bench.py: the byte counts behind its roofline line and its refusal of
more than one GPU.  No GPU is touched."""
import os
import subprocess
import sys

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
if ROOT not in sys.path:
    sys.path.insert(0, ROOT)

import bench          # noqa: E402
import workloads      # noqa: E402


def test_forward_launch_bytes_at_the_headline_shape():
    """700-128-128-20, T=128, B=256: the one forward launch reads the raster (1 byte per element)
    and the three rounded weight matrices (2 bytes), writes V (4) and S (1) of both layers and
    the readout's currents, trace and current gradients (4 bytes per padded class each)."""
    wl = workloads.CONFIGS["shd_ff128"]
    M = 128 * 256
    expect = M * 700 + 2 * (700 * 128 + 128 * 128 + 128 * 20) + 2 * M * 128 * 5 + 3 * M * 24 * 4
    assert expect == 74534912
    assert bench.forward_chain(wl, 1) == ([1, 2], True)
    assert bench.algorithmic_bytes(wl, "lif_forward", 1) == expect


def test_scan_and_weight_gradient_bytes_at_the_headline_shape():
    wl = workloads.CONFIGS["shd_ff128"]
    M = 128 * 256
    # reverse scans read the current gradients above (hi/lo words, padded columns) and V, write dI
    assert bench.algorithmic_bytes(wl, "lif_reverse", 2) == M * (24 * 4 + 128 * 8)
    assert bench.algorithmic_bytes(wl, "lif_reverse", 1) == M * (128 * 4 + 128 * 8)
    # weight gradients: spikes below (1 byte) and current gradients (4) of every layer, dW written
    expect = (M * 700 + M * 128 * 4 + 700 * 128 * 4) + (M * 128 + M * 128 * 4 + 128 * 128 * 4) + \
             (M * 128 + M * 20 * 4 + 128 * 20 * 4)
    assert bench.algorithmic_bytes(wl, "weight_grad", 0) == expect


def test_which_layers_run_as_one_forward_launch():
    """Mirrors the library's rule: feed-forward layers of at most 1024 neurons (fan-in too); pairs of at
    most 128; the readout rides along below 128 neurons and at most 32 padded classes."""
    cfg = workloads.CONFIGS
    assert bench.forward_chain(cfg["table1_ff512"], 1) == ([1], False)
    assert bench.forward_chain(cfg["wide_ff1024"], 2) == ([2], False)
    assert bench.forward_chain(cfg["deep_rec2048"], 2) == ([], False)
    assert bench.forward_chain(cfg["shd_rec128"], 1) == ([], False)
    assert bench.forward_chain(cfg["tiny_ff"], 1) == ([1], True)                    # fp32 products
    assert bench.forward_chain(cfg["shd_ff128"].scaled(precision="fp32"), 1) == ([1, 2], True)
    assert bench.forward_chain(cfg["shd_ff128"].scaled(sizes=(203, 121, 70, 33)), 1) == ([1, 2], False)
    five = cfg["shd_ff128"].scaled(sizes=(70, 64, 128, 128, 20), recurrent=(False,) * 3, beta=(0.9,) * 4)
    assert bench.forward_chain(five, 1) == ([1], False) and bench.forward_chain(five, 2) == ([2, 3], True)
    long = cfg["table1_ff512"].scaled(T=300, B=16)                                  # few samples of many steps
    assert bench.runs_whole(long, 1) and not bench.runs_whole(long.scaled(B=15), 1)
    steep = dict(adapt_decay=(0.9, 0.9), adapt_step=(0.2, 0.2))
    assert bench.forward_chain(cfg["shd_ff128"].scaled(**steep), 1) == ([1], False)
    assert bench.forward_chain(cfg["shd_ff128"].scaled(T=257, **steep), 1) == ([], False)
    assert not bench.runs_whole(cfg["shd_ff128"].scaled(adapt_decay=(0.9, 0.9), adapt_step=(float("inf"),) * 2), 1)


def test_reverse_launches_that_form_their_own_spike_gradients():
    cfg = workloads.CONFIGS
    assert all(bench.reverse_forms_ds(cfg["shd_ff128"].scaled(precision=p), l) for p in ("bf16", "fp32") for l in (1, 2))
    assert bench.reverse_forms_ds(cfg["shd_ff128"].scaled(sizes=(203, 130, 70, 11)), 1)
    assert not bench.reverse_forms_ds(cfg["table1_ff512"], 1) and bench.reverse_forms_ds(cfg["table1_ff512"], 2)
    few = cfg["shd_ff128"].scaled(precision="fp32", T=300, B=31)                    # six products below 128 columns
    assert not bench.reverse_forms_ds(few, 1) and bench.reverse_forms_ds(few.scaled(B=32), 1) and bench.reverse_forms_ds(few, 2)


def test_operations_of_a_pair_of_recurrent_layers():
    """Two recurrent layers of few neurons share a launch per direction, which also takes the product between them."""
    wl = workloads.CONFIGS["shd_rec128"]
    M = 128 * 256
    assert bench.recurrent_pair(wl, 1) and not bench.recurrent_pair(wl, 2)
    for kernel in ("rlif_forward", "rlif_reverse"):
        assert bench.method_flops(wl, kernel, 1) == 2 * M * 3 * 128 * 128
        assert bench.method_flops(wl.scaled(precision="fp32"), kernel, 1) == 2 * M * 128 * 128
        assert bench.method_flops(wl.scaled(sizes=(700, 168, 168, 20)), kernel, 1) == 2 * M * 168 * 168


def test_launch_bytes_of_fp32_products():
    """Three planes of the weights (2 bytes each); everything else as with rounded weights."""
    wl = workloads.CONFIGS["shd_ff128"].scaled(precision="fp32")
    M = 128 * 256
    weights = 700 * 128 + 128 * 128 + 128 * 20
    assert bench.algorithmic_bytes(wl, "lif_forward", 1) == M * 700 + 6 * weights + 2 * M * 128 * 5 + 3 * M * 24 * 4
    assert bench.algorithmic_bytes(wl, "lif_forward", 1, packed=True) == M // 8 * 700 + 6 * weights + 2 * M * 128 * 5 + 3 * M * 24 * 4
    assert bench.method_flops(wl, "lif_forward", 1) == 2 * M * weights


def test_more_than_one_gpu_is_refused():
    r = subprocess.run([sys.executable, os.path.join(ROOT, "bench.py"), "--gpus", "2"], capture_output=True, text=True,
                       timeout=120)
    assert r.returncode != 0
    assert "ONE GPU" in r.stderr and r.stdout.strip() == ""
