"""64-row tiles, whose K/V scan is walked in two halves at once: the edges of the halves and of each kernel's range of lengths."""
import math

import numpy as np
import pytest
import torch

from paper_2601_16032_amd import binding, workloads

from .util import assert_close

pytestmark = pytest.mark.gpu

# one tile to ten, odd and even, with a last tile of one row, of most, and of all 64
LENGTHS = [1, 64, 65, 100, 128, 129, 191, 192, 193, 256, 257, 320, 383, 448, 511, 513, 640]


def run(Q, K, V, scale, causal, order):
    """One workgroup per XCD: every other query tile of a head comes backward in sawtooth order."""
    var = binding.variant(kv_halves=2, slots_per_domain=1)
    O = binding.attn_fwd_variant(Q.cuda(), K.cuda(), V.cuda(), scale=scale, causal=causal, scan_order=order, o_dtype=torch.float32, variant=var)
    torch.cuda.synchronize()
    return O.double().cpu().numpy()


@pytest.mark.parametrize("causal", [False, True])
@pytest.mark.parametrize("dtype", ["f16", "bf16"])
@pytest.mark.parametrize("d", [64, 128])
def test_lengths_around_the_halves(d, dtype, causal):
    from oracle import attn_oracle
    for N in LENGTHS:
        Q, K, V = workloads.make_random(1, 8, N, d, dtype, seed=5000 + N)
        for scale in (1.0 / math.sqrt(d), -2.0):      # (the second raises the reference maximum again and again)
            want = attn_oracle.attention(Q, K, V, scale, causal=causal)
            for order in ("cyclic", "sawtooth"):
                assert_close(run(Q, K, V, scale, causal, order), want, f"N={N} d={d} {dtype} causal={causal} {order} {scale}")


@pytest.mark.parametrize("causal", [False, True])
@pytest.mark.parametrize("d", [64, 128])
def test_lengths_around_the_last_short_scan(d, causal):
    """Up to 64 K/V tiles a scan is short: the kernels on both sides, against the oracle on some rows."""
    from oracle import attn_oracle
    for N in (4032, 4095, 4096, 4097, 4160):
        Q, K, V = workloads.make_random(1, 1, N, d, "bf16", seed=6000 + N)
        scale = 1.0 / math.sqrt(d)
        rows = [0, 31, 32, 63, 64, N // 2, N - 65, N - 64, N - 1]
        want = attn_oracle.attention(Q, K, V, scale, causal=causal, rows=rows)[0, 0]
        for order in ("cyclic", "sawtooth"):
            assert_close(run(Q, K, V, scale, causal, order)[0, 0][rows], want, f"N={N} d={d} causal={causal} {order}")


@pytest.mark.parametrize("dtype", ["f16", "bf16"])
def test_masked_infinities_stay_where_they_are(dtype):
    """Infinite keys from `cut` on spoil no row before them, NaN values from `cut` on no row above their own 64-row tile (behind the mask, 0 times
    such a value is no number): those rows come out as without them, bit for bit."""
    for d in (64, 128):
        for cut in (1, 64, 100, 192, 300):
            Q, K, V = workloads.make_random(1, 8, 321, d, dtype, seed=7000 + cut)
            K2, V2 = K.clone(), V.clone()
            K2[:, :, cut:], V2[:, :, cut:] = float("inf"), float("nan")
            for order in ("cyclic", "sawtooth"):
                clean = run(Q, K, V, 0.1, True, order)
                assert np.isfinite(clean).all()
                for name, got, rows in (("K", run(Q, K2, V, 0.1, True, order), cut), ("V", run(Q, K, V2, 0.1, True, order), cut // 64 * 64)):
                    assert rows > 0 or (name, cut) == ("V", 1)
                    assert (clean[:, :, :rows] == got[:, :, :rows]).all(), f"{name} cut={cut} d={d} {dtype} {order}"
                    assert not np.isfinite(got[:, :, cut:]).any(), f"{name} cut={cut} d={d} {dtype} {order}"
