"""Row sums of the probabilities: every key of a row counts once, and no other row's keys do."""
import math

import pytest
import torch

from paper_2601_16032_amd import binding, workloads

from .util import SHARED_HEADS, SHARED_ROW_SUMS

pytestmark = pytest.mark.gpu

# one variant per scan: 64 query rows, 128 with a compute unit to each workgroup and with several workgroups to one, and (d = 128 only) 256
TILES = {"halves": dict(kv_halves=2), "rows32": dict(kv_halves=1, rows_per_wavefront=32),
         "shared": dict(kv_halves=1, rows_per_wavefront=32, launch="auto"), "rows64": dict(rows_per_wavefront=64)}
HEADS = {"shared": SHARED_HEADS}
LENGTHS = {"shared": SHARED_ROW_SUMS}


def run(Q, K, V, causal, tile):
    O = binding.attn_fwd_variant(Q.cuda(), K.cuda(), V.cuda(), scale=1.0 / math.sqrt(Q.shape[-1]), causal=causal, scan_order="cyclic",
                                 o_dtype=torch.float32, variant=binding.variant(**TILES[tile]))
    torch.cuda.synchronize()
    return O.cpu()


@pytest.mark.parametrize("causal", [False, True])
@pytest.mark.parametrize("dtype", ["f16", "bf16"])
@pytest.mark.parametrize("d,tile", [(64, "halves"), (64, "rows32"), (128, "halves"), (128, "rows32"), (128, "rows64"), (64, "shared"), (128, "shared")])
def test_every_key_counts_once(d, tile, dtype, causal):
    check(d, tile, dtype, causal, HEADS.get(tile, 8), LENGTHS.get(tile, (1, 63, 64, 65, 128, 191, 256, 321, 640)))


@pytest.mark.parametrize("causal", [False, True])
@pytest.mark.parametrize("dtype", ["f16", "bf16"])
@pytest.mark.parametrize("d", [64, 128])
def test_every_key_counts_once_in_long_scans_of_64_rows(d, dtype, causal):
    """Beyond 64 K/V tiles a scan in two halves runs in kernels of its own: an odd and an even number of tiles, and a ragged last one."""
    check(d, "halves", dtype, causal, 1, (4160, 4161, 4224))


def check(d, tile, dtype, causal, heads, lengths):
    for N in lengths:
        Q, K, V = workloads.make_random(1, heads, N, d, dtype, seed=9000 + N)
        # V = 1: the weighted sum and the row sum add the same rounded probabilities, each in binary32 in an order of its own
        O = run(Q, K, torch.ones_like(V), causal, tile)
        assert (O - 1.0).abs().max().item() <= 2.0 * (N + 8) * 2.0 ** -24, f"N={N}"
        # one row that is no number, between rows that stay as they are: 2^-9 for probabilities rounded to binary16 on another reference maximum
        bad = N // 2
        clean = run(Q, K, V, causal, tile)
        Q2 = Q.clone()
        Q2[:, :, bad] = float("nan")
        got = run(Q2, K, V, causal, tile)
        others = [r for r in range(N) if r != bad]
        assert got[:, :, bad].isnan().all(), f"N={N}"
        assert torch.allclose(got[:, :, others], clean[:, :, others], rtol=0.0, atol=2.0 ** -9 * V.float().abs().max().item()), f"N={N}"
