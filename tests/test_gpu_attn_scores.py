"""The prompt-phase attention tile where its running maximum matters: scores that grow along the
sequence (a new maximum in most key blocks), scores that differ by hundreds (one key carries a row),
and equal ones, over sequence ends and cache ends that cut a block of 64 keys anywhere."""
import math

import pytest
import torch

import inputs
import oracle
import paper_2305_13450_amd as ds
from gpu_util import TOL_BF16, TOL_FP16, row_err, run_attn_chain

pytestmark = pytest.mark.gpu


def _scaled(shape, seq, heads, dtype):
    t = inputs.attention(seq, 256, heads, 128, 64, seed=7, dtype=dtype)
    X = t["X"].float()
    if shape == "growing":
        X *= torch.linspace(0.2, 3.0, seq)[:, None]
    elif shape == "falling":
        X *= torch.linspace(3.0, 0.2, seq)[:, None]
    elif shape == "dominated":
        X *= 8.0
    elif shape == "equal":
        X[:] = X[0]
    t["X"] = X.to(dtype)
    return t


# Output and weights are rounded to 16 bits once each: 2^-9 of the largest of 128 elements (3.5 RMS of a
# random row) is 7e-3, and a row's weights, each off by up to 2^-9, add 1e-3 times 4 standard
# deviations: 2e-2 covers both; fp16 rounds to an eighth of that, 4e-3 is its bound throughout the suite.
@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float16])
@pytest.mark.parametrize("tile", [ds.TILE_128x192, ds.TILE_128x192_DEEP])   # two and four blocks in LDS
@pytest.mark.parametrize("seq", [1 * 64 + 1, 2 * 128, 3 * 128 - 1, 449, 640])
@pytest.mark.parametrize("shape", ["growing", "falling", "dominated", "equal"])
def test_rows_whatever_the_scores(shape, seq, tile, dtype):
    heads = 2
    t = _scaled(shape, seq, heads, dtype)
    print(f"attn scores {shape} seq={seq} tile={tile} {dtype}", flush=True)
    for split in (1, 0):
        pol = ds.SyncPolicy(ds.TILESYNC, ksplit=split)
        QKV, T, _ = run_attn_chain(t["X"], t["Wqkv"], t["Wo"], 1, seq, heads, pol, ds.MODE_FUSED, tile=tile)
        assert pol.status().timed_out == 0
        pol.destroy()
        ref = oracle.causal_attention(inputs.to_f64(QKV.cpu()), 1, seq, heads, 128)
        assert row_err(T, ref) <= (TOL_BF16 if dtype == torch.bfloat16 else TOL_FP16)


@pytest.mark.parametrize("dtype,tol", [(torch.bfloat16, TOL_BF16), (torch.float16, TOL_FP16)])
@pytest.mark.parametrize("tile", [ds.TILE_AUTO, ds.TILE_64x64, ds.TILE_128x192, ds.TILE_128x192_DEEP])
@pytest.mark.parametrize("seq,cached", [(300, 700), (300, 77), (257, 63), (640, 1)])
def test_cache_ends_inside_a_key_block(seq, cached, tile, dtype, tol):
    # A tile's last key block runs past its last query into rows it has not waited for.  They are masked,
    # but 0 x NaN is NaN, and a line read before its producer has posted would be stale for the next
    # query block: buffers start as NaN, are used again with other inputs, and a producer tile of the
    # second row tile posts late.
    heads = 2
    grid_x = -(-3 * heads * 128 // ds.tile_shape(tile)[1]) if tile else 4
    kv = inputs.kv_cache(1, cached, heads, 128, seed=cached, dtype=dtype)
    Kc, Vc = kv["Kc"].cuda(), kv["Vc"].cuda()
    print(f"cache end seq={seq} cached={cached} tile={tile} {dtype}", flush=True)
    QKV, T, Y = (torch.full((seq, n), float("nan"), dtype=dtype, device="cuda") for n in (3 * heads * 128, heads * 128, 64))
    for split in (1, 0):
        pol = ds.SyncPolicy(ds.TILESYNC, ksplit=split, delay_tile=2 * grid_x, delay_iters=20000)
        for seed in (1, 2):
            t = inputs.attention(seq, 256, heads, 128, 64, seed=seed, dtype=dtype)
            ds.dep_gemm_chain(t["X"].cuda(), t["Wqkv"].t().contiguous().cuda(), QKV, t["Wo"].t().contiguous().cuda(), Y, pol,
                              mode=ds.MODE_FUSED, mid=ds.MID_CAUSAL_ATTN, tile=tile, T=T, batch=1, seq=seq, heads=heads,
                              head_dim=128, k_cache=Kc, v_cache=Vc)
            torch.cuda.synchronize()
            ref = oracle.cached_attention(inputs.to_f64(QKV.cpu()), inputs.to_f64(kv["Kc"]), inputs.to_f64(kv["Vc"]), 1, seq, heads, 128)
            assert row_err(T, ref) <= tol
        assert pol.status().timed_out == 0
        pol.destroy()


@pytest.mark.parametrize("dtype,bits", [(torch.bfloat16, 8), (torch.float16, 11)])
@pytest.mark.parametrize("tile", [ds.TILE_128x192, ds.TILE_128x192_DEEP])
def test_weights_are_summed_in_32_bits(tile, dtype, bits):
    # QKV = X: key 0 has the largest score and the only value (ones), every other key the same weight p and no value,
    # so row i is 1 / (1 + i p) and shows the sum of the weights alone.  p is chosen half way between two
    # 16-bit numbers: a sum over rounded weights is off by half of a last place, and the result by more than the
    # half that its own rounding may take.
    seq, a = 640, 16.0
    best = max((d / 64 for d in range(1, 32)), key=lambda d: abs(_last_places(_weight(a, d), bits) % 1.0 - 0.5) * -1)
    p = _weight(a, best)
    assert abs(_last_places(p, bits) % 1.0 - 0.5) < 0.1
    X = torch.zeros(seq, 384)
    X[:, 0] = a
    X[0, 128], X[1:, 128] = 1.0, 1.0 - best
    X[0, 256:] = 1.0
    pol = ds.SyncPolicy(ds.TILESYNC, ksplit=1)
    QKV, T, _ = run_attn_chain(X.to(dtype), torch.eye(384).to(dtype), torch.zeros(128, 64).to(dtype), 1, seq, 1, pol, ds.MODE_FUSED, tile=tile)
    assert pol.status().timed_out == 0
    pol.destroy()
    assert torch.equal(QKV.cpu().float(), X)
    ref = 1.0 / (1.0 + p * torch.arange(seq, dtype=torch.float64))[:, None]
    half = torch.exp2(torch.floor(torch.log2(ref)) - bits)
    # fp32: up to 640 additions and an exponential of 1e-7 each, 1e-5 with room
    assert ((T.cpu().double() - ref).abs() <= half + 1e-5 * ref).all()


def _weight(a, d):
    return math.exp(-a * d / math.sqrt(128.0))


def _last_places(x, bits):
    return x * 2.0 ** (bits - 1 - math.floor(math.log2(x)))
