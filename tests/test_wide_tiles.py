"""256-row tiles (64 query rows per wavefront, head dimension 128): the edges of the scan's pipeline, and what may not reach a row."""
import math

import pytest
import torch

from paper_2601_16032_amd import binding, workloads

from .util import assert_close

pytestmark = pytest.mark.gpu

# lengths around whole numbers of K/V tiles up to more than the four buffers, with a last tile of one row, of most, and of all 64; two
# query tiles and three
LENGTHS = [1, 64, 127, 128, 129, 191, 193, 256, 257, 319, 321, 384, 447, 449, 512, 513, 577, 640]
KINDS = ["f16", "bf16", "bf16-workspace"]


def call(kind):
    return binding.attn_fwd_workspace if kind == "bf16-workspace" else binding.attn_fwd_variant


@pytest.mark.parametrize("causal", [False, True])
@pytest.mark.parametrize("kind", KINDS)
def test_lengths_around_the_pipeline(kind, causal):
    """Every element against the oracle, walked up and down (one workgroup per XCD: every other query tile of a head comes backward)."""
    from oracle import attn_oracle
    dtype = kind.split("-")[0]
    var = binding.variant(rows_per_wavefront=64, slots_per_domain=1)
    for N in LENGTHS:
        Q, K, V = workloads.make_random(1, 8, N, 128, dtype, seed=3000 + N)
        scale = 1.0 / math.sqrt(128)
        want = attn_oracle.attention(Q, K, V, scale, causal=causal)
        for order in ("cyclic", "sawtooth"):
            O = call(kind)(Q.cuda(), K.cuda(), V.cuda(), scale=scale, causal=causal, scan_order=order, o_dtype=torch.float32, variant=var)
            torch.cuda.synchronize()
            assert_close(O.double().cpu().numpy(), want, f"N={N} {kind} causal={causal} {order}")


@pytest.mark.parametrize("causal", [False, True])
@pytest.mark.parametrize("kind", KINDS)
def test_no_other_rows_are_read(kind, causal):
    """K and V of every other head, and of the rows before the first head and behind the last one, once hold ordinary values and once NaN
    and infinities: the heads in between come out the same bit for bit."""
    dtype = kind.split("-")[0]
    guard, H = 256, 24
    bad = ((torch.arange(H) % 2) ^ (torch.arange(H) // 8 % 2)).bool().cuda()
    for N in (1, 65, 129, 321, 577):
        Q, K, V = (t.cuda() for t in workloads.make_random(1, H, N, 128, dtype, seed=8000 + N))

        def inside(t, fill):
            room = torch.full((guard + H * N + guard, 128), fill, dtype=t.dtype, device="cuda")
            room[guard:-guard] = t.reshape(-1, 128)
            return room[guard:-guard].view(t.shape)
        for order, kw in (("cyclic", {}), ("sawtooth", dict(slots_per_domain=1))):
            var = binding.variant(rows_per_wavefront=64, **kw)
            outs = []
            for k_fill, v_fill in ((0.0, 0.0), (float("nan"), float("inf"))):
                Kg, Vg = inside(K, k_fill), inside(V, v_fill)
                if k_fill != 0.0:
                    Kg[:, bad], Vg[:, bad] = k_fill, v_fill
                outs.append(call(kind)(Q, Kg, Vg, scale=1.0 / math.sqrt(128), causal=causal, scan_order=order, o_dtype=torch.float32, variant=var))
            torch.cuda.synchronize()
            assert torch.isfinite(outs[0]).all() and torch.equal(outs[0][:, ~bad], outs[1][:, ~bad]), f"N={N} {order}"


@pytest.mark.parametrize("dtype", ["f16", "bf16"])
def test_masked_infinities_stay_where_they_are(dtype):
    """Causal: an infinite key spoils no row before it, an infinite value no row above its own 64-row tile (behind the mask, 0 times an
    infinite value is no number), walked up, where the tiles behind a wavefront's rows come last, and down, where they come first.
    A NaN query row spoils itself alone."""
    N, H = 1000, 8
    Q, K, V = workloads.make_random(1, H, N, 128, dtype, seed=91)
    var = binding.variant(rows_per_wavefront=64, slots_per_domain=1)       # tiles 3, 1 of a head up, 2, 0 down under the sawtooth order

    def run(Q, K, V, order):
        O = binding.attn_fwd_variant(Q.cuda(), K.cuda(), V.cuda(), scale=0.09, causal=True, scan_order=order, o_dtype=torch.float32, variant=var)
        torch.cuda.synchronize()
        return O
    for order in ("cyclic", "sawtooth"):
        clean = run(Q, K, V, order)
        assert torch.isfinite(clean).all()
        for bad in (70, 200, 330, 460, 600, 900, 999):
            Kb, Vb, Qb = K.clone(), V.clone(), Q.clone()
            Kb[0, :, bad, 0], Vb[0, :, bad], Qb[0, :, bad] = float("inf"), float("inf"), float("nan")
            assert torch.equal(run(Q, Kb, V, order)[:, :, :bad], clean[:, :, :bad]), (order, bad)
            above = bad // 64 * 64
            assert torch.equal(run(Q, K, Vb, order)[:, :, :above], clean[:, :, :above]), (order, bad)
            O, rest = run(Qb, K, V, order), [r for r in range(N) if r != bad]
            assert torch.isnan(O[0, :, bad]).all() and torch.equal(O[:, :, rest], clean[:, :, rest]), (order, bad)
