"""Which workgroups of a direct causal launch start first, which launches are direct, and what computes them.

The order in which workgroups start is no part of the schedule: every workgroup computes and records what the schedule oracle lists for
its number.  The CPU tests compile schedule.h, the header that the library is built from."""
import math
import os
import subprocess

import pytest
import torch

from paper_2601_16032_amd import binding, workloads

from .util import SHARED_EVEN, assert_close, oracle_inputs

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def ask(tmp_path_factory):
    """(heads, N, d, bf16, query rows per tile) -> per causal direct launch with one tile per workgroup, longest first or (last argument) as
    the caller's variant names it: what computes it (A, S or P: the 32x32x16 kernel, the 16x16x32 one without and with precedence), chunks
    per XCD, workgroups per chunk, and the workgroups of XCD 3 in the order in which they start."""
    d = tmp_path_factory.mktemp("order")
    (d / "order.cpp").write_text("""#include <stdio.h>
#include "schedule.h"
using namespace sawattn;
int main() {
    int heads, N, d, bf16, tile_q, named;
    while (scanf("%d %d %d %d %d %d", &heads, &N, &d, &bf16, &tile_q, &named) == 6) {
        Schedule s = launch_schedule(heads, N, d, true, tile_q, kLaunchGrid, kDecodeDomain, 0, 1);
        if (!named) start_longest_first(s, d, true);
        printf("%c %d %d", !default_shared_kernel(s, d, true, bf16) ? 'A' : default_phase_priority(s, d, true) ? 'P' : 'S',
               s.chunks_per_domain, s.units_per_chunk);
        for (int block = 3; block < s.grid; block += kDomains) printf(" %d", workgroup_of_block(s, block));
        puts("");
    }
}
""")
    subprocess.run(["g++", "-std=c++17", "-Wall", "-I", os.path.join(ROOT, "paper_2601_16032_amd", "csrc"), str(d / "order.cpp"),
                    "-o", str(d / "order")], check=True, capture_output=True)

    def run(cases, named=False):
        text = "\n".join(" ".join(str(int(x)) for x in c + (named,)) for c in cases)
        lines = subprocess.run([str(d / "order")], input=text, check=True, capture_output=True, text=True).stdout.splitlines()
        out = []
        for line in lines:
            f = line.split()
            out.append((f[0], int(f[1]), int(f[2]), [int(x) for x in f[3:]]))
        return out
    return run


# launches that start longest first, and those that lose by it (3 or 5 workgroups to each of many chunks) or have one workgroup to a chunk
LONGEST_FIRST = [(32, 4096, 128, 0, 128), (97, 1100, 128, 0, 128), (9, 1000, 64, 0, 128), (5, 129, 64, 1, 128), (128, 4096, 64, 0, 128),
                 (17, 12000, 64, 0, 128), (24, 2600, 64, 0, 64), (11, 1400, 128, 0, 64), (40, 3968, 64, 1, 128), (102, 1500, 128, 1, 128),
                 (70, 2883, 128, 0, 128), (106, 2436, 128, 0, 128), (126, 3500, 128, 1, 128), (127, 2700, 64, 0, 128), (121, 11904, 128, 0, 128)]
IN_ORDER = [(1, 64, 64, 0, 128), (8, 100, 128, 0, 128), (107, 2880, 128, 0, 128), (103, 3000, 128, 0, 128), (110, 2176, 128, 1, 128)]
ORDER_CASES = LONGEST_FIRST + IN_ORDER


def test_blocks_are_a_permutation_of_the_workgroups_longest_first(ask):
    for case, (_, chunks, units, order) in zip(ORDER_CASES, ask(ORDER_CASES)):
        n = chunks * units
        assert sorted(order) == [8 * k + 3 for k in range(n)], case        # every workgroup of the XCD once, on its XCD
        slots = [(w // 8) // units for w in order], [(w // 8) % units for w in order]
        resident = 32 if case[2] == 128 else 64
        resident = resident if case[4] == 64 else (64 if case[2] == 128 else 96)
        if case in IN_ORDER:
            assert order == sorted(order), case
            continue
        # groups of consecutive chunks, one after the other, each of 3/2 loads at least unless there is only one; in a group the position
        # in the chunk (0 is the longest) never falls
        chunk, pos = slots
        starts = [i for i in range(1, n) if pos[i] < pos[i - 1]]
        groups = [range(a, b) for a, b in zip([0] + starts, starts + [n])]
        seen = []
        for g in groups:
            mine = sorted(set(chunk[i] for i in g))
            assert len(g) == len(mine) * units and mine == list(range(mine[0], mine[0] + len(mine))), case
            seen += mine
        assert seen == list(range(chunks)), case
        assert len(groups) == 1 or all(2 * len(g) >= 3 * resident for g in groups[:-1]), case


def test_a_direct_launch_that_is_named_starts_in_the_order_of_its_numbers(ask):
    """Alg. 3 as printed can be measured: only what attn_fwd picks by itself starts longest first."""
    for case, (_, chunks, units, order) in zip(ORDER_CASES, ask(ORDER_CASES, named=True)):
        assert order == [8 * k + 3 for k in range(chunks * units)], case


def test_what_computes_a_launch_whose_longest_workgroups_start_first(ask):
    """Both sides of every line, each the faster way when measured (to 1 %)."""
    by_hand = [     # (heads, N, d, bf16)
        ((5, 8191, 128, 0), "A"), ((10, 4376, 128, 0), "A"), ((6, 8960, 128, 1), "A"), ((50, 854, 128, 0), "S"), ((21, 2816, 128, 0), "S"),
        ((74, 640, 128, 0), "P"), ((33, 1536, 128, 1), "P"), ((5, 13824, 128, 0), "S"), ((10, 8038, 128, 1), "S"), ((32, 4096, 128, 0), "P"),
        ((13, 7457, 128, 0), "P"), ((12, 9117, 128, 0), "P"), ((17, 13184, 128, 0), "P"), ((24, 7936, 128, 0), "S"), ((24, 7168, 128, 0), "S"),
        ((27, 1792, 64, 1), "S"), ((37, 1672, 64, 1), "P"), ((12, 7168, 64, 1), "S"), ((5, 16965, 64, 1), "S"), ((64, 2048, 64, 0), "S"),
        ((40, 3968, 64, 1), "S"), ((20, 6784, 64, 1), "P"), ((14, 8381, 64, 0), "P"), ((32, 8192, 64, 0), "P"), ((104, 3507, 64, 0), "P"),
    ]
    got = [a[0] for a in ask([c + (128,) for c, _ in by_hand])]
    wrong = [(c, w, g) for (c, w), g in zip(by_hand, got) if w != g]
    assert not wrong, wrong


DIRECT = [     # (B, H, N, d, causal): the launch that attn_fwd picks
    # causal, one round per chunk: an odd number of rounds, an even one that does not fill the compute units evenly
    ((1, 24, 5000, 128, True), "grid"), ((1, 6, 16667, 128, True), "grid"), ((1, 24, 8192, 128, True), "grid"), ((1, 56, 8192, 128, True), "persistent"),
    ((1, 16, 4352, 128, True), "grid"), ((1, 16, 8000, 128, True), "grid"), ((1, 16, 8192, 128, True), "persistent"), ((1, 32, 7680, 128, True), "grid"),
    ((1, 32, 7808, 128, True), "persistent"), ((1, 16, 6144, 64, True), "grid"), ((1, 16, 7680, 64, True), "persistent"), ((1, 16, 9216, 64, True), "grid"),
    ((1, 16, 12288, 64, True), "persistent"), ((1, 32, 7680, 64, True), "grid"), ((1, 32, 8192, 64, True), "persistent"), ((1, 8, 10000, 64, True), "persistent"),
    # several rounds per chunk
    ((1, 16, 13440, 64, True), "grid"), ((1, 16, 23296, 64, True), "persistent"), ((8, 1, 32768, 64, True), "grid"), ((1, 8, 27008, 64, True), "persistent"),
    ((1, 16, 8960, 128, True), "grid"), ((1, 16, 14720, 128, True), "persistent"), ((1, 8, 17920, 128, True), "persistent"),
    ((1, 16, 8320, 128, False), "grid"), ((1, 8, 8320, 128, False), "persistent"), ((1, 16, 12544, 64, False), "grid"), ((1, 16, 24576, 64, False), "persistent"),
    ((1, 1, 131072, 64, False), "grid"), ((1, 8, 18432, 64, False), "persistent"), ((1, 8, 24576, 64, False), "persistent"),
    # exactly on the line (128 tiles on 96 places: 3/2), and a tile to either side
    ((1, 8, 16256, 64, False), "grid"), ((1, 8, 16384, 64, False), "grid"), ((1, 8, 16385, 64, False), "persistent"),
    # 64-row tiles
    ((1, 24, 2600, 64, True), "grid"), ((1, 16, 3000, 64, True), "grid"), ((1, 16, 3900, 64, True), "persistent"), ((1, 16, 2048, 64, True), "persistent"),
]


@pytest.mark.parametrize("shape,want", DIRECT)
def test_which_launches_are_direct(shape, want):
    info = binding.attn_fwd_launch_info(*shape)
    assert ["persistent", "grid"][info["launch"]] == want and info["tiles_per_workgroup"] == 1
    # a variant that names the launch, or the number of workgroups, gets what it names
    assert binding.attn_fwd_variant_launch_info(*shape, binding.variant(launch="persistent"))["launch"] == binding.LAUNCH_PERSISTENT
    assert binding.attn_fwd_variant_launch_info(*shape, binding.variant(launch="auto", slots_per_domain=7))["launch"] == binding.LAUNCH_PERSISTENT


SEVERAL_ROUNDS = [(1, 1, 131072, 64, False), (1, 16, 12544, 64, False), (8, 1, 32768, 64, True), (1, 2, 131072, 64, True), (1, 16, 13440, 64, True),
                  (1, 16, 8320, 128, False), (1, 16, 8960, 128, True), (1, 20, 27000, 64, True)]


@pytest.mark.parametrize("shape", SEVERAL_ROUNDS)
@pytest.mark.parametrize("order", ["cyclic", "sawtooth"])
def test_direct_launches_keep_the_scan_directions_of_the_rounds(shape, order):
    """A launch that is direct instead of persistent walks every tile the way the persistent launch does: under the sawtooth order the odd
    rounds go down.  A direct launch that the caller asks for has no rounds."""
    def tiles(**kw):
        trace, count = binding.attn_fwd_plan(*shape, scan_order=order, variant=binding.variant(kv_halves=1, **kw) if kw else None)
        return sorted(tuple(r) for wg in range(len(count)) for r in trace[wg, : int(count[wg])].tolist())
    assert binding.attn_fwd_launch_info(*shape)["launch"] == binding.LAUNCH_GRID
    got = tiles()
    assert got == tiles(launch="persistent", rows_per_wavefront=32)
    assert any(first > last for _, _, first, last in got) == (order == "sawtooth")
    assert all(first <= last for _, _, first, last in tiles(launch="grid", tiles_per_workgroup=1, rows_per_wavefront=32))


@pytest.mark.gpu
@pytest.mark.parametrize("H,N,d,dtype,causal", [(16, 12500, 64, "f16", False), (16, 13440, 64, "bf16", True), (20, 27000, 64, "f16", True)])
def test_direct_and_persistent_launches_give_the_same_bits(H, N, d, dtype, causal):
    """At d = 64 one kernel computes both launches, and no other order of summation may come from the launch."""
    assert binding.attn_fwd_launch_info(1, H, N, d, causal, dtype=dtype)["launch"] == binding.LAUNCH_GRID
    q, k, v = (t.cuda() for t in workloads.make_random(1, H, N, d, dtype, seed=900 + H))
    scale, O = 1.0 / math.sqrt(d), {}
    for order in ("cyclic", "sawtooth"):
        O[order] = binding.attn_fwd(q, k, v, scale=scale, causal=causal, scan_order=order, o_dtype=torch.float32)
        same = binding.attn_fwd_variant(q, k, v, scale=scale, causal=causal, scan_order=order, o_dtype=torch.float32,
                                        variant=binding.variant(launch="persistent", kv_halves=1))
        torch.cuda.synchronize()
        assert torch.equal(O[order], same), order
    assert not torch.equal(O["cyclic"], O["sawtooth"])


# Causal launches of every kernel and of one and two groups of chunks, and the plain ones that are direct now.
GPU_CASES = [
    (17, 2048, 128, "f16", True, "A"), (25, 1800, 128, "bf16", True, "S"), (35, 2100, 128, "f16", True, "P"), (97, 1100, 128, "bf16", True, "P"),
    (17, 3100, 128, "f16", True, "S"), (17, 2040, 64, "bf16", True, "S"), (49, 1100, 64, "f16", True, "P"), (64, 2000, 64, "bf16", True, "S"),
    (*SHARED_EVEN, 64, "f16", True, "S"), (*SHARED_EVEN, 64, "bf16", True, "S"), (*SHARED_EVEN, 128, "f16", True, "S"),
    (*SHARED_EVEN, 128, "bf16", True, "S"), (24, 2600, 64, "f16", True, None), (11, 1400, 128, "bf16", True, None), (24, 5000, 128, "f16", True, None), (16, 8300, 128, "bf16", False, None),
]


@pytest.mark.gpu
@pytest.mark.parametrize("H,N,d,dtype,causal,kernel", GPU_CASES)
def test_started_longest_first_computes_and_records_the_same(ask, H, N, d, dtype, causal, kernel):
    from oracle import attn_oracle, schedule_oracle as so
    if kernel:
        assert ask([(H, N, d, dtype == "bf16", 128)])[0][0] == kernel
    info = binding.attn_fwd_launch_info(1, H, N, d, causal, dtype=dtype)
    assert info["launch"] == binding.LAUNCH_GRID
    Q, K, V = workloads.make_random(1, H, N, d, dtype, seed=700 + H)
    q, k, v = Q.cuda(), K.cuda(), V.cuda()
    scale = 1.0 / math.sqrt(d)
    rows = sorted(set(list(range(0, N, 211)) + [1, 63, 64, 127, 128, N - 129, N - 65, N - 1]))
    heads = [0, H // 2, H - 1]
    want = attn_oracle.attention(Q[:, heads], K[:, heads], V[:, heads], scale, causal=causal, rows=rows)
    for order in ("cyclic", "sawtooth"):
        O, trace, count = binding.attn_fwd_variant(q, k, v, scale=scale, causal=causal, scan_order=order, o_dtype=torch.float32, trace=True)
        plain = binding.attn_fwd(q, k, v, scale=scale, causal=causal, scan_order=order, o_dtype=torch.float32)
        torch.cuda.synchronize()
        assert torch.equal(O, plain)
        assert_close(O.double().cpu().numpy()[:, heads][:, :, rows], want, f"{H} x {N}, {d} {dtype} {order}")
        trace, count = trace.cpu(), count.cpu()
        sched = so.schedule(1, H, N, causal, order, **oracle_inputs(info, d))
        assert trace.shape[0] == len(sched)
        for wg, recs in sched.items():
            assert [tuple(r) for r in trace[wg, : int(count[wg])].tolist()] == recs, f"workgroup {wg}"
