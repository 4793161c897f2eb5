"""Performance cases: the attention forward as a program calls it, from one tiny head to the largest workload.

The shapes are the five workloads of `paper_2601_16032_amd.workloads`, shapes of the package's own sweeps (short
heads, the paper's sequence-length and batch studies) and of its tests (ragged lengths, head counts that do not divide
over the eight XCDs).  A state is what a serving or prefill loop holds before the call: Q, K, V of one layer on the
GPU, the output buffer and, for the entry point that takes one, a workspace.  `draw` gives more cases of the same
ranges: 1..128 heads, sequences of 64..131072 rows, both head dimensions, element types, masks and scan orders.
"""
from __future__ import annotations

import math

import torch

from paper_2601_16032_amd import binding

_DTYPE = {"f16": torch.float16, "bf16": torch.bfloat16, "f32": torch.float32}


def _case(B, H, N, d, dtype, out, causal, order="sawtooth", entry="attn_fwd", gain=1.0, k_offset=0.0):
    return {"B": B, "H": H, "N": N, "d": d, "dtype": dtype, "out": out, "causal": causal, "order": order,
            "entry": entry, "gain": gain, "k_offset": k_offset}


def listed():
    def named(name, *args, **kw):
        return {"name": name, **_case(*args, **kw)}
    return [
        # workload 1: one short head, nothing but latency (a single request, a unit of a larger program)
        named("one_head_256", 1, 1, 256, 64, "f16", "f16", False),
        # workload 2: one layer of a small model at its full context, too small to fill the chip by itself
        named("layer_8x2048", 1, 8, 2048, 64, "f16", "f16", False),
        # a batch of short prompts, many heads each (the short-heads sweep)
        named("short_heads_128x512", 8, 16, 512, 128, "f16", "f16", False),
        # odd in everything: 42 heads (not a multiple of the XCDs), a length that is no multiple of a tile, causal
        named("ragged_42x1000", 2, 21, 1000, 64, "bf16", "f32", True),
        # an ordinary causal prefill of a 4K prompt
        named("prefill_32x4096", 1, 32, 4096, 128, "f16", "f16", True),
        # an encoder layer in bfloat16 throughout: 12 heads, ragged length, every key visible
        named("encoder_12x5000", 1, 12, 5000, 128, "bf16", "bf16", False, order="cyclic"),
        # workload 3: causal prefill in bfloat16, 8K context
        named("prefill_16x8192", 1, 16, 8192, 128, "bf16", "f32", True),
        # a 16K prefill whose caller lends scratch memory
        named("prefill_ws_32x16384", 1, 32, 16384, 128, "bf16", "f32", True, entry="attn_fwd_workspace"),
        # workload 4, the benchmark's headline shape
        named("full_32x16384", 1, 32, 16384, 128, "f16", "f16", False, gain=0.5),
        # the paper's batch study at head dimension 64, causal
        named("batch_8x32768", 8, 1, 32768, 64, "f16", "f16", True),
        # the paper's single long head at head dimension 64
        named("long_1x131072", 1, 1, 131072, 64, "f16", "f16", False, order="cyclic"),
        # workload 5: a full causal batch at 32K, the largest
        named("prefill_128x32768", 4, 32, 32768, 128, "bf16", "f32", True, k_offset=0.5),
    ]


_MOST_FLOPS = 4.0 * 128 * 32768.0 ** 2 * 128 / 2     # workload 5
_MOST_ELEMENTS = 128 * 32768 * 128


def draw(rng):
    """One more case: log-uniform head count and length, redrawn while it would cost more than workload 5."""
    while True:
        N = int(round(math.exp(rng.uniform(math.log(64), math.log(131072)))))
        if rng.random() < 0.4:                       # whole tiles are as common as ragged lengths
            N = max(64, N // 64 * 64)
        heads = int(round(math.exp(rng.uniform(0.0, math.log(128)))))
        B = rng.choice([b for b in (1, 2, 3, 4, 8) if heads % b == 0])
        d = rng.choice([64, 128])
        causal = rng.random() < 0.5
        if 4.0 * heads * float(N) * N * d / (2 if causal else 1) <= _MOST_FLOPS and heads * N * d <= _MOST_ELEMENTS:
            break
    dtype = rng.choice(["f16", "bf16"])
    return _case(B, heads // B, N, d, dtype, "f16" if dtype == "f16" else rng.choice(["f32", "bf16"]), causal,
                 order=rng.choice(["sawtooth", "sawtooth", "sawtooth", "cyclic"]),
                 entry="attn_fwd_workspace" if dtype == "bf16" and rng.random() < 0.25 else "attn_fwd",
                 gain=rng.choice([0.5, 1.0]), k_offset=rng.choice([0.0, 0.5]) if dtype == "bf16" else 0.0)


def prepare(case, seed):
    g = torch.Generator("cuda").manual_seed(int(seed))
    B, H, N, d = case["B"], case["H"], case["N"], case["d"]
    dt = _DTYPE[case["dtype"]]

    def normal():
        x = torch.randn((B, H, N, d), generator=g, device="cuda", dtype=torch.float32)
        return x.mul_(case["gain"]) if case["gain"] != 1.0 else x
    q = normal().to(dt)
    k = normal()
    if case["k_offset"]:                             # one common offset per head, as in workload 5
        k += torch.randn((B, H, 1, d), generator=g, device="cuda", dtype=torch.float32) * case["k_offset"]
    k = k.to(dt)
    v = normal().to(dt)
    state = {"q": q, "k": k, "v": v, "o": torch.empty((B, H, N, d), dtype=_DTYPE[case["out"]], device="cuda"),
             "scale": 1.0 / math.sqrt(d), "causal": case["causal"], "order": case["order"], "workspace": None,
             "entry": case["entry"]}
    if case["entry"] == "attn_fwd_workspace":
        need, _ = binding.attn_fwd_workspace_bytes(B, H, N, d, case["causal"], None, case["dtype"])
        if need:
            state["workspace"] = torch.empty(need, dtype=torch.uint8, device="cuda")
    return state


def run(state):
    if state["entry"] == "attn_fwd_workspace":
        return binding.attn_fwd_workspace(state["q"], state["k"], state["v"], state["o"], scale=state["scale"],
                                          causal=state["causal"], scan_order=state["order"],
                                          workspace=state["workspace"])
    return binding.attn_fwd(state["q"], state["k"], state["v"], state["o"], scale=state["scale"],
                            causal=state["causal"], scan_order=state["order"])


def work(case):
    """Q, K, V read once and O written once; two products of 2 flops per multiply-add, halved under the causal mask."""
    elements = case["B"] * case["H"] * case["N"] * case["d"]
    flops = 4.0 * elements * case["N"] / (2 if case["causal"] else 1)
    return {"bytes": elements * (3 * 2 + (4 if case["out"] == "f32" else 2)), "flops": flops}


def tolerance(case):
    """Binary16 probabilities and 32-bit sums: measured 1.6e-4 (32-bit output) to 3.0e-4 (binary16 output) from the
    64-bit result, 1.7e-3 where the output is rounded to bfloat16; about four times that."""
    return {"rel": 7e-3 if case["out"] == "bf16" else 1.2e-3}


def exact(case, seed):
    """Softmax(Q K^T scale) V in 64 bits from the same inputs, a panel of query rows of one head at a time."""
    s = prepare(case, seed)
    N, d = case["N"], case["d"]
    q, k, v = (s[n].reshape(-1, N, d) for n in ("q", "k", "v"))
    out = torch.empty(q.shape, dtype=torch.float64, device="cuda")
    rows = max(1, min(N, (1 << 28) // N))
    for h in range(q.shape[0]):
        kt, vh = k[h].double().t().contiguous(), v[h].double()
        for r0 in range(0, N, rows):
            r1 = min(N, r0 + rows)
            n = r1 if case["causal"] else N          # keys any row of the panel sees
            p = torch.mm(q[h, r0:r1].double(), kt[:, :n].contiguous()).mul_(s["scale"])
            if case["causal"]:
                p.masked_fill_(torch.arange(n, device="cuda")[None, :] > torch.arange(r0, r1, device="cuda")[:, None],
                               -math.inf)
            p.sub_(p.amax(dim=1, keepdim=True)).exp_()
            out[h, r0:r1] = torch.mm(p, vh[:n]) / p.sum(dim=1, keepdim=True)
    return out.reshape(case["B"], case["H"], N, d)
