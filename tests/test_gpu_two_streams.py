"""The two-stream form (side launches, draws by compare-and-swap), which a chain takes when the tiles of its
earlier stages do not all fit on the GPU at once, and chains of several policies on the GPU together."""
import pytest
import torch

import inputs
import oracle
import paper_2305_13450_amd as ds
from gpu_util import TOL_BF16, rel_err

pytestmark = pytest.mark.gpu


def _gemm():
    # 64 x 16 = 1024 producer tiles on 512 slots
    M, K1, N1, N2 = 4096, 128, 1024, 256
    ts = [inputs.mlp(M, K1, N1, N2, seed=s) for s in (1, 2)]
    W1t, W2t = ts[0]["W1"].t().contiguous().cuda(), ts[0]["W2"].t().contiguous().cuda()
    Xs = [t["X"].cuda() for t in ts]
    H, Y = (torch.empty((M, n), dtype=torch.bfloat16, device="cuda") for n in (N1, N2))

    def run(i, pol, mode):
        ds.dep_gemm_chain(Xs[i], W1t, H, W2t, Y, pol, mode=mode, tile=ds.TILE_64x64)
        return [H, Y]
    return run, ds._gemm_desc(Xs[0], W1t, H, W2t, Y, ds.MID_GELU, ds.TILE_64x64), 2


def _attention():
    # 48 x 16 = 768 tiles of QKV, 64 of attention
    seq, heads, K1, N2 = 1024, 8, 128, 128
    ts = [inputs.attention(seq, K1, heads, 128, N2, seed=s) for s in (1, 2)]
    Wq, Wo = ts[0]["Wqkv"].t().contiguous().cuda(), ts[0]["Wo"].t().contiguous().cuda()
    Xs = [t["X"].cuda() for t in ts]
    QKV, T, Y = (torch.empty((seq, n), dtype=torch.bfloat16, device="cuda") for n in (3 * heads * 128, heads * 128, N2))
    kw = dict(T=T, batch=1, seq=seq, heads=heads, head_dim=128)

    def run(i, pol, mode):
        ds.dep_gemm_chain(Xs[i], Wq, QKV, Wo, Y, pol, mode=mode, mid=ds.MID_CAUSAL_ATTN, tile=ds.TILE_64x64, **kw)
        return [QKV, T, Y]
    return run, ds._gemm_desc(Xs[0], Wq, QKV, Wo, Y, ds.MID_CAUSAL_ATTN, ds.TILE_64x64, **kw), 3


def _convolutions():
    # four stages of 196 row tiles: 588 tiles before the last stage
    shape = (4, 56, 56, 64)
    g = torch.Generator().manual_seed(5)
    xs = [torch.randn(shape, generator=g).to(torch.bfloat16).cuda() for _ in range(2)]
    ws = [(torch.randn((64, 3, 3, 64), generator=g) * (2 / 576) ** 0.5).to(torch.bfloat16).cuda() for _ in range(4)]
    outs = [torch.empty(shape, dtype=torch.bfloat16, device="cuda") for _ in range(4)]

    def run(i, pol, mode):
        ds.dep_conv_chain_n(xs[i], ws, outs, pol, mode=mode, tile=ds.TILE_64x64)
        return outs
    return run, ds._conv_n_desc(xs[0], ws, outs, ds.TILE_64x64), 4


@pytest.mark.parametrize("kw", [{}, dict(delay_tile=1, delay_iters=300), dict(delay_tile=100, delay_iters=300), dict(delay_tile=530, delay_iters=300),
                                dict(flags=ds.FLAG_REVERSE_ORDER), dict(flags=ds.FLAG_NO_REORDER)])
@pytest.mark.parametrize("kind", [ds.ROWSYNC, ds.TILESYNC, ds.STRIDEDSYNC])
@pytest.mark.parametrize("chain", [_gemm, _attention, _convolutions])
def test_side_launches_give_the_bits_of_stream_sync(chain, kind, kw):
    # late posts, reversed draws, and inputs that change on the same buffers from chain to chain (a stale
    # line of the intermediate would give the other answer)
    if chain is _gemm and kind == ds.STRIDEDSYNC:
        kw = dict(kw, stride=4)
    run, desc, stages = chain()
    print(f"two streams {chain.__name__} kind={kind} {kw}", flush=True)
    pol = ds.SyncPolicy(kind, **kw)
    assert ds.launch_form(desc, pol, ds.MODE_FINE) == (stages, False)
    base = ds.SyncPolicy(kind, **{k: v for k, v in kw.items() if k == "stride"})
    want = []
    for i in (0, 1):
        want.append([t.clone() for t in run(i, base, ds.MODE_STREAMSYNC)])
    assert not torch.equal(want[0][-1], want[1][-1])
    got = []
    for it in range(8):                                                  # back to back, no host sync in between
        got.append([t.clone() for t in run(it & 1, pol, ds.MODE_FUSED if it == 5 else ds.MODE_FINE)])
    torch.cuda.synchronize()
    for it, g in enumerate(got):
        assert all(torch.equal(a, b) for a, b in zip(g, want[it & 1])), it
    assert pol.status().timed_out == 0
    base.destroy()
    pol.destroy()


@pytest.mark.parametrize("tiles", [(ds.TILE_64x192, ds.TILE_64x64), (ds.TILE_128x128_DEEP, ds.TILE_64x128)])
@pytest.mark.parametrize("ksplit", [2, 8])
def test_split_tiles_of_a_side_launch_chain_after_chain(tiles, ksplit):
    # the producer, on the side stream, may still be running when the next chain begins on the same words (M = 61: one row of tiles,
    # of which every part finishes a slice)
    M, K1, N1, N2 = 61, 1024, 3072, 256
    ts = [inputs.mlp(M, K1, N1, N2, seed=s) for s in (1, 2)]
    W1t, W2t = ts[0]["W1"].t().contiguous().cuda(), ts[0]["W2"].t().contiguous().cuda()
    Xs = [t["X"].cuda() for t in ts]
    H, Y = (torch.empty((M, n), dtype=torch.bfloat16, device="cuda") for n in (N1, N2))
    print(f"side launch with split tiles {tiles} ksplit={ksplit}", flush=True)
    for kind in (ds.ROWSYNC, ds.TILESYNC):
        pol = ds.SyncPolicy(kind, ksplit=ksplit)
        assert ds.launch_form(ds._gemm_desc(Xs[0], W1t, H, W2t, Y, ds.MID_GELU, tiles), pol, ds.MODE_FINE) == (2, False)

        def run(i, mode):
            ds.dep_gemm_chain(Xs[i], W1t, H, W2t, Y, pol, mode=mode, tile=tiles)
            return H.clone(), Y.clone()
        want = [run(i, ds.MODE_STREAMSYNC) for i in (0, 1)]
        assert not torch.equal(want[0][1], want[1][1])
        got = [run(it & 1, ds.MODE_FINE) for it in range(40)]             # no host sync in between
        torch.cuda.synchronize()
        for it, (h, y) in enumerate(got):
            assert torch.equal(h, want[it & 1][0]) and torch.equal(y, want[it & 1][1]), it
        assert pol.status().timed_out == 0
        pol.destroy()


def test_chains_of_several_policies_at_once():
    # Each of these chains could hold every slot by itself.  In the default mode they draw from the
    # queues, which progress whatever the others hold.
    t = inputs.mlp(256, 1024, 4096, 1024, seed=7)
    ref = oracle.gemm_chain(inputs.to_f64(t["X"]), inputs.to_f64(t["W1"]), inputs.to_f64(t["W2"]), oracle.ACT_GELU)[1]
    X, W1t, W2t = t["X"].cuda(), t["W1"].t().contiguous().cuda(), t["W2"].t().contiguous().cuda()
    chains = []
    for kind in (ds.ROWSYNC, ds.TILESYNC, ds.ROWSYNC, ds.TILESYNC):
        H, Y = (torch.full((256, n), float("nan"), dtype=X.dtype, device="cuda") for n in (4096, 1024))
        pol = ds.SyncPolicy(kind)
        assert ds.launch_form(ds._gemm_desc(X, W1t, H, W2t, Y, ds.MID_GELU, ds.TILE_AUTO), pol, ds.MODE_FINE) == (1, False)
        chains.append((pol, torch.cuda.Stream(), H, Y))
        ds.dep_gemm_chain(X, W1t, H, W2t, Y, pol)                          # (the first call may grow the policy's scratch buffer)
    torch.cuda.synchronize()
    for _ in range(20):
        for pol, stream, H, Y in chains:
            stream.wait_stream(torch.cuda.current_stream())
            ds.dep_gemm_chain(X, W1t, H, W2t, Y, pol, stream_producer=stream)
    torch.cuda.synchronize()
    for pol, _, H, Y in chains:
        assert pol.status().timed_out == 0 and rel_err(Y, ref) <= TOL_BF16
        assert torch.equal(Y, chains[0][3])
        pol.destroy()
