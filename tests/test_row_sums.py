"""Row sums of the probabilities: every key of a row counts once, and no other row's keys do."""
import math

import pytest
import torch

from paper_2601_16032_amd import binding, workloads

pytestmark = pytest.mark.gpu

# one variant per tile height: 64, 128 and (d = 128 only) 256 query rows
TILES = {"halves": dict(kv_halves=2), "rows32": dict(kv_halves=1, rows_per_wavefront=32), "rows64": dict(rows_per_wavefront=64)}


def run(Q, K, V, causal, tile):
    O = binding.attn_fwd_variant(Q.cuda(), K.cuda(), V.cuda(), scale=1.0 / math.sqrt(Q.shape[-1]), causal=causal, scan_order="cyclic",
                                 o_dtype=torch.float32, variant=binding.variant(**TILES[tile]))
    torch.cuda.synchronize()
    return O.cpu()


@pytest.mark.parametrize("causal", [False, True])
@pytest.mark.parametrize("dtype", ["f16", "bf16"])
@pytest.mark.parametrize("d,tile", [(64, "halves"), (64, "rows32"), (128, "halves"), (128, "rows32"), (128, "rows64")])
def test_every_key_counts_once(d, tile, dtype, causal):
    for N in (1, 63, 64, 65, 128, 191, 256, 321, 640):
        Q, K, V = workloads.make_random(1, 8, N, d, dtype, seed=9000 + N)
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
