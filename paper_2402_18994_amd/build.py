"""Compile the HIP library for gfx950 in-tree (hipcc cross-compiles without a GPU)."""
import concurrent.futures
import os
import subprocess
import sys
import tempfile

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
OUT = os.path.join(HERE, "libsnn_hip.so")

FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC",
         # keep the compiler from forming packed fp32 VALU instructions
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
         "-Wall", "-Wno-unused-function"]
# translation unit -> flags of its own
# (The speed of the short launches depends on where their code lies: the feed-forward step runs the same instructions
# in, us at T = B = 128 / T = 128, B = 256 of 700-128-128-20: 65.1 / 76.9 where the linker puts them, 63.5 / 76.4 at
# multiples of 1 KiB; multiples of 4 and 64 KiB are no better.  The reverse launches of narrow layers at multiples of 4 KiB against 1 KiB,
# everything else the same, both builds in turn, twice: T = 128, B = 256 85.4, 85.9 and 85.8, 86.8, with fp32-exact products 104.1,
# 103.6 and 104.3, 103.8, packed at T = 256 136.1, 136.1 and 138.2, 138.3.  These are properties of a build: a change elsewhere
# that moves the kernels is worth as much, either way.)
UNITS = {"snn_api.hip": ["-Xarch_device", "-falign-functions=1024"],
         "layer_forward.hip": ["-Xarch_device", "-falign-functions=1024"],
         "layer_forward_wide.hip": ["-Xarch_device", "-falign-functions=1024"],
         "layer_reverse.hip": ["-Xarch_device", "-falign-functions=4096"],
         "layer_reverse_wide.hip": ["-Xarch_device", "-falign-functions=1024"],
         "rlif_wide.hip": [],
         # results of MFMAs in ordinary vector registers (the time loops read them at once)
         "rlif_pair.hip": ["-mllvm", "-amdgpu-mfma-vgpr-form"],
         "rlif_tile.hip": ["-mllvm", "-amdgpu-mfma-vgpr-form"]}


def _run(cmd, verbose: bool) -> None:
    if verbose:
        print(" ".join(cmd), flush=True)
    res = subprocess.run(cmd, capture_output=True, text=True)
    noise = "packed-fp32-ops"
    err = "\n".join(l for l in res.stderr.splitlines() if noise not in l)
    if res.returncode != 0:
        raise RuntimeError("hipcc failed:\n" + err)
    if verbose and err.strip():
        print(err, file=sys.stderr)


def build(verbose: bool = False) -> str:
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    extra = os.environ.get("SNN_EXTRA_FLAGS", "").split()
    with tempfile.TemporaryDirectory() as tmp, concurrent.futures.ThreadPoolExecutor(len(UNITS)) as pool:
        objs = {u: os.path.join(tmp, u + ".o") for u in UNITS}
        jobs = [pool.submit(_run, [hipcc] + FLAGS + UNITS[u] + extra + ["-c", "-o", objs[u], os.path.join(CSRC, u)], verbose)
                for u in UNITS]
        for j in jobs:
            j.result()
        _run([hipcc, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", OUT] + list(objs.values()), verbose)
    return OUT


if __name__ == "__main__":
    print(build(verbose=True))
