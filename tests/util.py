"""Shared helpers for the tests (comparison metrics and launch facts only; no attention arithmetic)."""
import glob
import os
import re
import shutil
import subprocess

import numpy as np

MAX_ABS_TOL = 2e-3     # stated tolerance of the benchmark definition, fp16/bf16 inputs
REL_L2_TOL = 1e-3


def errors(got, want):
    got = np.asarray(got, dtype=np.float64)
    want = np.asarray(want, dtype=np.float64)
    assert got.shape == want.shape, (got.shape, want.shape)
    assert np.all(np.isfinite(got)), "non-finite values in the GPU output"
    diff = got - want
    max_abs = float(np.abs(diff).max()) if diff.size else 0.0
    denom = float(np.sqrt((want * want).sum()))
    rel_l2 = float(np.sqrt((diff * diff).sum()) / denom) if denom > 0 else 0.0
    return max_abs, rel_l2


def assert_close(got, want, what=""):
    max_abs, rel_l2 = errors(got, want)
    assert max_abs <= MAX_ABS_TOL and rel_l2 <= REL_L2_TOL, (
        f"{what}: max-abs {max_abs:.3e} (tol {MAX_ABS_TOL}), rel-L2 {rel_l2:.3e} (tol {REL_L2_TOL})")
    return max_abs, rel_l2


# Workgroups of one XCD that run at the same time, by (head dimension, query rows per workgroup tile): 32 CUs times
# the workgroups a CU holds (three at d = 64: 32 KiB LDS and at most 168 registers each; two at d = 128; one with
# 256-row tiles, which take 128 KiB LDS and 512 registers per wavefront; with 64-row tiles -- the two halves of the
# K/V scan at once, twice the LDS of a 128-row tile -- two at d = 64 and one at d = 128).  Listed here by hand: the
# schedule oracle takes it as an input and the library's own figure is compared with it.
RESIDENT_PER_XCD = {(64, 128): 96, (128, 128): 64, (128, 256): 32, (64, 64): 64, (128, 64): 32}


def oracle_inputs(info, d, variant_kw=None):
    """Inputs of oracle.schedule_oracle for a launch of the library: the tile height and the kind of launch the
    library reports (its choices are pinned case by case in test_host_logic.py), the hand-listed resident count, and
    the variant's work decode."""
    kw = dict(variant_kw or {})
    out = {k: v for k, v in kw.items() if k in ("launch", "decode", "tiles_per_workgroup")}
    if kw.get("launch", "auto") == "auto":      # left open: what the library reports (persistent if it says nothing)
        out["launch"] = ("persistent", "grid")[info.get("launch", 0)]
    if out["launch"] == "grid" and "tiles_per_workgroup" not in out and "tiles_per_workgroup" in info:
        out["tiles_per_workgroup"] = info["tiles_per_workgroup"]
    out["tile_q"] = info["tile_q"]
    out["resident"] = kw.get("slots_per_domain") or RESIDENT_PER_XCD[(d, info["tile_q"])]
    if kw.get("launch", "auto") == "auto" and out["launch"] == "grid":     # walked as in the persistent launch it stands in for
        out["turn_after"] = out["resident"]
    return out


# Short heads that make the kernel for compute units shared by workgroups run (33 workgroups and more per XCD; too many heads
# for a halved scan), and lengths at which, launched one or two tiles per workgroup, they reach every build of it: both head
# dimensions and input types, without a mask, and under the mask with (one tile) and without (two) precedence by phase (two tiles at d = 128 with 2, 4 or
# 8 workgroups per head, as at 129..256 and 385..512 rows, is left to the other kernel there).
SHARED_HEADS = 264
SHARED_LENGTHS = [1, 63, 64, 65, 128, 129, 200, 321, 577]
# (heads, rows) whose causal launch, left open, reaches the build without precedence at both head dimensions: all 49 workgroups of an XCD at
# once, the last tile of a head one of 65 rows.  (With 264 heads the lengths above have it from two tiles per workgroup.)
SHARED_EVEN = (56, 833)
# Lengths at which SHARED_HEADS run on that kernel without exception, launched as the library chooses, for its row sums.
SHARED_ROW_SUMS = [1, 63, 64, 65, 128, 321, 577]


def llvm_tool(name, *args):
    """What one of the LLVM tools that come with the compiler of the library prints."""
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    tool = subprocess.run([hipcc, f"-print-prog-name={name}"], check=True, capture_output=True, text=True).stdout.strip()
    return subprocess.run([tool, *args], check=True, capture_output=True, text=True).stdout


def device_code(into):
    """The code object inside the built library, unpacked into the directory `into`."""
    from paper_2601_16032_amd import build as hip_build
    lib = shutil.copy(hip_build.LIB_PATH, os.path.join(into, "lib.so"))
    llvm_tool("llvm-objdump", "--offloading", lib)
    path, = glob.glob(lib + "*gfx950")
    return path


def device_listing(into):
    """The assembly of the built library's kernels."""
    return llvm_tool("llvm-objdump", "-d", "--mcpu=gfx950", device_code(into)).splitlines()


def kernel_bodies(listing):
    """{kernel: [(instruction, index of the instruction it may branch to, or None)]}, names as in the source."""
    mangled, kernels = None, {}
    for line in listing:
        head = re.match(r"[0-9a-f]+ <(\w+)>:", line)
        if head:
            mangled = head.group(1)
            kernels[mangled] = []
            continue
        code = re.match(r"\t(\S.*?)\s*// ([0-9A-F]+): [0-9A-F ]+(?:<\w+\+0x([0-9a-f]+)>)?", line)
        if code and mangled:
            kernels[mangled].append((code.group(1), int(code.group(2), 16), code.group(3)))
    names = subprocess.run(["c++filt", *kernels], check=True, capture_output=True, text=True).stdout.splitlines()
    out = {}
    for name, body in zip(names, kernels.values()):
        at = {address: i for i, (_, address, _) in enumerate(body)}
        out[name] = [(text, at[body[0][1] + int(to, 16)] if to else None) for text, _, to in body]
    return out
