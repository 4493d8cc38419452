"""The work that a user of this library has it do, as cases that can be timed and compared.

A case names a network (`sizes`, one `recurrent` flag per spiking layer), a batch (`T` steps of `B`
samples), the options of the network (`precision`, `surrogate`, `loss`, `learn_beta`, `adaptive`,
`packed`: the raster packed along time) and what is done with it:

  train         one training step: forward, backward, SGD step, nothing read back in between
  evaluate      forward, then the loss and the logits on the host, as an accuracy count needs them
  weight_grad   dW = S^T G alone, on the caller's tensors (the entry point that allocates nothing)

Rasters and weights have the statistics of workloads.py: channel rates drawn once, independent
Bernoulli spikes, N(0, gain / sqrt(fan_in)) weights.  The gain is 3 as in the tests, so that hidden
layers fire at a few percent, as those of a trained network do (at gain 1 they are nearly silent); in
networks with a recurrent layer, whose own spikes come back to it, it is 1.5.
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2402_18994_amd import SNN, weight_grad_static

LEARNING_RATE = {"max": 1e-3, "integral": 1e-6}      # (the integral loss sums the readout over time)
RECURRENT_GAIN = 0.5
DECAY = 0.95
SLOPES = {"superspike": 25.0, "arctan": 2.0, "sigmoid": 4.0, "triangular": 1.0, "boxcar": 1.0, "ste": 1.0}


def _case(name, T, B, sizes, recurrent="", do="train", precision="bf16", surrogate="superspike", loss="max",
          learn_beta=False, adaptive=False, packed=False):
    case = dict(do=do, T=T, B=B, sizes=sizes, recurrent=recurrent or "-".join("0" * (sizes.count("-") - 1)),
                precision=precision, surrogate=surrogate, loss=loss, learn_beta=learn_beta, adaptive=adaptive,
                packed=packed)
    return dict(name=name, **case) if name else case


def listed():
    return [
        # the smallest network of the benchmark list, all in fp32: a step is launches and latency
        _case("tiny_fp32", 32, 16, "100-64-10", precision="fp32", surrogate="arctan"),
        # the headline network: the ordinary training step
        _case("ff128", 128, 256, "700-128-128-20"),
        # the same in the arithmetic of the paper's own timing runs
        _case("ff128_fp32", 128, 256, "700-128-128-20", precision="fp32"),
        # twice as many time steps, the raster in the paper's storage format
        _case("ff128_packed", 256, 256, "700-128-128-20", packed=True),
        # recurrent hidden layers: a time loop that no batching over steps shortens
        _case("rec128", 128, 256, "700-128-128-20", "1-1"),
        # the paper's wider timing run
        _case("ff512", 256, 256, "700-512-512-20"),
        # wide layers: products of the size that fills the matrix units
        _case("ff1024", 256, 512, "700-1024-1024-20"),
        # deep, long, wide and recurrent: the largest of the benchmark list
        _case("deep_rec2048", 512, 128, "700-2048-2048-2048-20", "1-0-0", surrogate="arctan"),
        # sizes that are multiples of nothing, one layer recurrent, decays trained, the paper's integral loss
        _case("ragged", 101, 51, "203-130-70-11", "1-0", surrogate="sigmoid", loss="integral", learn_beta=True),
        # adaptive firing thresholds with trained decays
        _case("adaptive256", 128, 128, "700-256-256-20", surrogate="triangular", learn_beta=True, adaptive=True),
        # a batch of the validation set: loss and logits
        _case("evaluate", 256, 256, "700-128-128-20", do="evaluate"),
        # one weight gradient on the caller's own tensors, at the headline's first layer
        _case("weight_grad", 128, 256, "700-128", do="weight_grad", precision="fp32"),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _width(rng, lo, hi):
    """A layer width: as often a round one as any other."""
    n = _log(rng, lo, hi)
    return max(64, n // 64 * 64) if rng.random() < 0.5 else n


def _flops(T, B, sizes, recurrent):
    pairs = [(a * b) for a, b in zip(sizes, sizes[1:])] + [n * n for n, r in zip(sizes[1:], recurrent) if r]
    return 6.0 * T * B * sum(pairs)


def draw(rng):
    do = rng.choices(("train", "evaluate", "weight_grad"), (12, 3, 1))[0]
    precision = rng.choices(("bf16", "fp32"), (3, 1))[0]
    T, B = _log(rng, 16, 512), _log(rng, 4, 512)
    if rng.random() < 0.5:
        T, B = max(16, T // 16 * 16), max(4, B // 8 * 8)
    if do == "weight_grad":
        sizes = [4 * _log(rng, 8, 256), 4 * _log(rng, 4, 256)]
        return _case(None, T, B, "%d-%d" % tuple(sizes), do=do, precision="fp32")
    wide = 512 if precision == "fp32" else 2048
    channels = rng.choice((700, 700, rng.randrange(40, 1000)))
    hidden = [_width(rng, 16, wide)]
    for _ in range(rng.choice((0, 1, 1, 2))):
        hidden.append(hidden[0] if rng.random() < 0.6 else _width(rng, 16, wide))
    sizes = [channels] + hidden + [rng.choice((10, 20, 20, rng.randrange(2, 40)))]
    adaptive = rng.random() < 0.15
    recurrent = [int(not adaptive and i == 0 and rng.random() < 0.3) for i in range(len(hidden))]
    if recurrent[0] and rng.random() < 0.5:
        recurrent = [1] * len(hidden)
    # no more than the largest listed case: its operations (fp32 products take several passes each),
    # its steps of a wide recurrent layer, and a tensor's limit of 2 GiB
    most = _flops(512, 128, [700, 2048, 2048, 2048, 20], [1, 0, 0]) / (6 if precision == "fp32" else 1)
    while _flops(T, B, sizes, recurrent) > most or T * B * (max(sizes) + 8) * 4 >= 1 << 30:
        if B > 4:
            B = max(4, B // 2)
        else:
            T = T // 2
    if max([n for n, r in zip(hidden, recurrent) if r], default=0) > 128:
        T, B = min(T, 256 // sum(recurrent)), min(B, 128)
    # (a surrogate that does not fall off away from the threshold lets the gradient of a recurrent
    # layer grow from step to step until it overflows)
    surrogate = rng.choice(("superspike", "superspike", "arctan", "sigmoid") + (() if any(recurrent) else ("triangular", "boxcar", "ste")))
    return _case(None, T, B, "-".join(map(str, sizes)), "-".join(map(str, recurrent)), do=do, precision=precision,
                 surrogate=surrogate, loss=rng.choice(("max", "max", "integral")),
                 learn_beta=do == "train" and rng.random() < 0.2, adaptive=adaptive, packed=rng.random() < 0.25)


def network(case):
    sizes = [int(n) for n in case["sizes"].split("-")]
    return sizes, [r == "1" for r in case["recurrent"].split("-")] if len(sizes) > 2 else []


def inputs(case, seed):
    """Raster, labels and initial parameters of a case, drawn on the GPU from the seed."""
    gen = torch.Generator(device="cuda").manual_seed(seed)
    sizes, recurrent = network(case)
    T, B = case["T"], case["B"]
    # (at least as many input spikes per step as the 700 channels at 0.5 to 4 % give a small network)
    rates = torch.empty(sizes[0], device="cuda").uniform_(0.005, 0.04, generator=gen) * max(1.0, min(4.0, 250.0 / sizes[0]))
    x = torch.empty(T, B, sizes[0], dtype=torch.uint8, device="cuda")
    for t in range(T):
        x[t] = torch.rand(B, sizes[0], device="cuda", generator=gen) < rates

    def normal(rows, cols, deviation):
        return (torch.randn(rows, cols, device="cuda", generator=gen) * deviation).cpu().numpy()

    gain = 1.5 if any(recurrent) else 3.0
    W = [normal(a, b, gain / math.sqrt(a)) for a, b in zip(sizes, sizes[1:])]
    R = [normal(n, n, RECURRENT_GAIN * gain / math.sqrt(n)) if r else None for n, r in zip(sizes[1:], recurrent)]
    labels = torch.randint(0, sizes[-1], (B,), device="cuda", generator=gen).to(torch.int32)
    betas = [(0.9 + 0.09 * torch.rand(n, device="cuda", generator=gen)).cpu().numpy() for n in sizes[1:]]
    return x, labels, W, R, betas


def pack_time(x):
    """numpy.packbits(x, axis=0) on the GPU: eight steps a byte, the first in the highest bit."""
    T = x.shape[0]
    pad = torch.zeros((-T % 8,) + tuple(x.shape[1:]), dtype=x.dtype, device=x.device)
    groups = torch.cat([x, pad]).view(-1, 8, *x.shape[1:])
    out = torch.zeros_like(groups[:, 0])
    for k in range(8):
        out |= groups[:, k] << (7 - k)
    return out.contiguous()


def build(case, W, R, betas):
    """The network object a program keeps over its training run."""
    sizes, recurrent = network(case)
    L = len(sizes) - 1
    snn = SNN(case["T"], case["B"], sizes, recurrent, [DECAY] * L, 1.0, case["surrogate"], SLOPES[case["surrogate"]],
              case["precision"], W, R, loss=case["loss"], learn_beta=case["learn_beta"],
              adapt_decay=[0.9] * (L - 1) if case["adaptive"] else None,
              adapt_step=[0.2] * (L - 1) if case["adaptive"] else None)
    if case["learn_beta"]:                       # decays of a network in training differ from neuron to neuron
        for l in range(L):
            snn.set_tensor("beta", l + 1, betas[l])
    return snn


def _in_workspace(snn, name, layer):
    """The tensor as the library keeps it: a view of the workspace that the caller handed over.

    Parameters, their gradients and the per-sample losses are contiguous there, each at a 256-byte
    boundary; the place is found by the values (the largest one first, then all of them)."""
    value = torch.from_numpy(snn.get_tensor(name, layer)).to(snn.device)
    flat = value.reshape(-1)
    words = snn.workspace[: snn.workspace.numel() // 256 * 256].view(torch.float32)
    at = int(flat.abs().argmax())
    for block in (words[at % 64::64] == flat[at]).nonzero().reshape(-1).tolist():
        start = block * 64 + at % 64 - at
        if start >= 0 and start + flat.numel() <= words.numel() and torch.equal(words[start:start + flat.numel()], flat):
            return words[start:start + flat.numel()].view(value.shape)
    raise LookupError("%s of layer %d is not in the workspace" % (name, layer))


def prepare(case, seed):
    T, B = case["T"], case["B"]
    sizes, recurrent = network(case)
    if case["do"] == "weight_grad":
        gen = torch.Generator(device="cuda").manual_seed(seed)
        K, N = sizes
        rates = torch.empty(K, device="cuda").uniform_(0.005, 0.04, generator=gen)
        spikes = (torch.rand(T * B, K, device="cuda", generator=gen) < rates).to(torch.uint8)
        grads = torch.randn(T * B, N, device="cuda", generator=gen) / B
        return {"do": case["do"], "args": (spikes, grads, torch.empty(K, N, device="cuda"))}
    x, labels, W, R, betas = inputs(case, seed)
    if case["packed"]:
        x = pack_time(x)
    snn = build(case, W, R, betas)
    state = {"do": case["do"], "snn": snn, "x": x, "labels": labels, "forward": snn.forward_packed if case["packed"] else snn.forward}
    if case["do"] == "train":
        # the gradients of the first batch show where the library keeps its results
        state["forward"](x, labels, want_loss=False)
        snn.backward()
        layers = range(1, len(sizes))
        out = {"loss_per_sample": _in_workspace(snn, "loss_per_sample", 0)}
        for name in ("weight", "grad_w") + (("beta", "grad_beta") if case["learn_beta"] else ()):
            out[name] = [_in_workspace(snn, name, l) for l in layers]
        for name in ("rweight", "grad_r"):
            out[name] = [_in_workspace(snn, name, l) for l in layers if l < len(sizes) - 1 and recurrent[l - 1]]
        state["out"], state["lr"] = out, LEARNING_RATE[case["loss"]]
    return state


def run(state):
    if state["do"] == "weight_grad":
        weight_grad_static(*state["args"])
        return state["args"][2]
    snn = state["snn"]
    if state["do"] == "evaluate":
        loss = state["forward"](state["x"], state["labels"])
        return {"loss": loss, "logits": snn.get_tensor("logits")}
    state["forward"](state["x"], state["labels"], want_loss=False)
    snn.backward()
    snn.sgd_step(state["lr"])
    return state["out"]


def work(case):
    """Raster, labels and parameters read once, results written once; one multiplication and one
    addition per term of a product (forward, and for the gradients of weights and of spikes), about
    twenty operations per neuron and step beside them."""
    sizes, recurrent = network(case)
    T, B = case["T"], case["B"]
    M = T * B
    if case["do"] == "weight_grad":
        K, N = sizes
        return {"bytes": M * K + 4 * M * N + 4 * K * N, "flops": 2 * M * K * N}
    products = [a * b for a, b in zip(sizes, sizes[1:])]
    own = [n * n for n, r in zip(sizes[1:], recurrent) if r]
    raster = -(-T // 8) * B * sizes[0] if case["packed"] else M * sizes[0]
    parameters = sum(products) + sum(own)
    if case["do"] == "evaluate":
        return {"bytes": raster + 4 * B + 4 * parameters + 4 * B * sizes[-1],
                "flops": 2 * M * parameters + 6 * M * sum(sizes[1:])}
    # weights read, written back, and their gradients written
    return {"bytes": raster + 8 * B + 12 * parameters,
            "flops": 2 * M * (3 * parameters - products[0]) + 20 * M * sum(sizes[1:])}


def tolerance(case):
    """About four times what the same pass differs by when every sum is taken in another order (units
    and samples permuted, or the other kernels of the same step), measured over the listed cases
    and 100 drawn ones.

    Mostly that is 1e-7 to 1e-5.  Now and then a potential lies so close to the threshold that its
    spike falls the other way; the sample's later steps then differ, and so do the gradients it
    adds to: 8e-3 of dW^1, 0.17 at one element, with fp32 products; 5e-4 and 0.04 with rounded
    weights, whose sums in fp32 are nearly exact.  A product alone, against 64 bits: 1.2e-7 and 7e-7."""
    if case["do"] == "weight_grad":
        return {"rel": 5e-7, "max": 3e-6}
    if case["precision"] == "fp32":
        return {"rel": 3e-2, "max": 0.7}
    return {"rel": 2e-3, "max": 0.15}
