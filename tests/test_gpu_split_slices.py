"""Tiles split along K of which every part finishes a slice of the rows: slices of odd and no rows, every number of
parts, and parts that end before others of their tile have been started.  Inputs are small whole numbers whose
sums are exact in fp32 and in bf16, so every result is compared bit for bit; the activations, the gated product, fp16, packed
weights and convolutions are compared with the oracle, and between the modes bit for bit."""
import pytest
import torch

import inputs
import oracle
import paper_2305_13450_amd as ds
from gpu_util import TOL_BF16, TOL_FP16, TOL_MID, mid_err, rel_err, run_gemm_chain

pytestmark = pytest.mark.gpu

MODES = [ds.MODE_FUSED, ds.MODE_FINE, ds.MODE_STREAMSYNC, ds.MODE_PLAIN]
SLICED = [ds.TILE_64x192, ds.TILE_128x192_DEEP, ds.TILE_128x128_DEEP, ds.TILE_256x128, ds.TILE_128x256]


def whole_numbers(M, K1, N1, N2):
    g = torch.Generator().manual_seed(M)
    X = (torch.rand((M, K1), generator=g) < 0.1).float() * torch.randint(-2, 3, (M, K1), generator=g)
    W1 = torch.randint(-2, 3, (K1, N1), generator=g).float()
    W2 = (torch.rand((N1, N2), generator=g) < 0.05).float() * torch.randint(-1, 2, (N1, N2), generator=g)
    H = X @ W1
    assert H.abs().max() < 256                    # whole numbers that bf16 holds
    Y = H.double() @ W2.double()
    assert Y.abs().max() < 2 ** 24                # ... and fp32 sums
    return [t.to(torch.bfloat16) for t in (X, W1, W2)], H, Y.to(torch.bfloat16)


@pytest.mark.parametrize("tile", SLICED)
@pytest.mark.parametrize("M", [1, 4, 5, 31, 66, 129, 252])
def test_every_number_of_parts_and_rows(M, tile):
    ops, H, Y = whole_numbers(M, 1536, 768, 264)
    for ksplit in (2, 3, 4, 6, 8):
        print(f"slices M={M} tile={tile} ksplit={ksplit}", flush=True)
        for kind in (ds.ROWSYNC, ds.TILESYNC):
            pol = ds.SyncPolicy(kind, ksplit=ksplit, flags=ds.FLAG_COUNT)
            for mode in MODES:
                h, y = run_gemm_chain(*ops, pol, mode, mid=ds.MID_NONE, tile=tile)
                assert torch.equal(h.cpu().float(), H) and torch.equal(y.cpu(), Y)
            st = pol.status()
            tm, tn = ds.tile_shape(tile)
            assert st.timed_out == 0 and st.posts == 3 * -(-M // tm) * -(-768 // tn)   # one post per tile and mode with hooks
            pol.destroy()


@pytest.mark.parametrize("tile,M", [(ds.TILE_64x192, 61), (ds.TILE_128x192_DEEP, 117)])
def test_parts_that_end_before_others_start(tile, M):
    # 64 column tiles in eight parts are 512 workgroups on a chip that holds 256: with tiles named by the block
    # index the first parts of every tile end before the last have been started, and leave their slices behind
    ops, H, Y = whole_numbers(M, 1024, 12288, 72)
    print(f"late parts tile={tile}", flush=True)
    rows, cols = ds.tile_shape(tile)
    n_tiles = 12288 // cols
    for flags, modes in ((0, MODES), (ds.FLAG_HW_ORDER, [ds.MODE_STREAMSYNC, ds.MODE_FUSED])):
        pol = ds.SyncPolicy(ds.ROWSYNC, ksplit=8, flags=flags | ds.FLAG_TRACE)
        for mode in modes:
            for _ in range(2):
                h, y = run_gemm_chain(*ops, pol, mode, mid=ds.MID_NONE, tile=tile)
                assert torch.equal(h.cpu().float(), H) and torch.equal(y.cpu(), Y)
            if mode != ds.MODE_PLAIN:
                # a part that had ended when another of its tile was handed out cannot have waited for it
                recs = pol.read_trace(8 * n_tiles)
                assert sorted((r.tx, r.ty) for r in recs) == [(x, z) for x in range(n_tiles) for z in range(8)]
                late = sum(min(r.t_end for r in recs if r.tx == x) < max(r.t_start for r in recs if r.tx == x) for x in range(n_tiles))
                assert late > 0
        assert pol.status().timed_out == 0
        pol.destroy()


@pytest.mark.parametrize("tile", SLICED)
def test_the_spin_limit_is_for_dependency_waits(tile):
    # one launch after the other: no tile waits for a producer, and the parts of a tile wait for one another however small the limit is
    ops, H, Y = whole_numbers(129, 1536, 768, 264)
    print(f"spin limit tile={tile}", flush=True)
    for ksplit in (2, 8):
        pol = ds.SyncPolicy(ds.TILESYNC, ksplit=ksplit, spin_limit=1)
        for mode in (ds.MODE_PLAIN, ds.MODE_STREAMSYNC):
            for _ in range(3):
                h, y = run_gemm_chain(*ops, pol, mode, mid=ds.MID_NONE, tile=tile)
                assert pol.status().timed_out == 0
                assert torch.equal(h.cpu().float(), H) and torch.equal(y.cpu(), Y)
        pol.destroy()


@pytest.mark.parametrize("tile", [ds.TILE_64x192, ds.TILE_128x128_DEEP, ds.TILE_256x128])
def test_parts_wait_out_a_sibling_that_waits_for_a_late_tile(tile):
    # One tile of the producer posts a millisecond or two late.  The consumer parts that read it wait (a few thousand polls, inside
    # the limit), their siblings wait for them, and every row is written.
    ops, H, Y = whole_numbers(129, 1536, 768, 264)
    print(f"late sibling tile={tile}", flush=True)
    for ksplit in (2, 4):
        pol = ds.SyncPolicy(ds.TILESYNC, ksplit=ksplit, spin_limit=40000, delay_tile=1, delay_iters=400)
        for mode in (ds.MODE_FUSED, ds.MODE_FINE):
            h, y = run_gemm_chain(*ops, pol, mode, mid=ds.MID_NONE, tile=tile)
            assert pol.status().timed_out == 0
            assert torch.equal(h.cpu().float(), H) and torch.equal(y.cpu(), Y)
        pol.destroy()


@pytest.mark.parametrize("tile", [ds.TILE_128x128_DEEP, ds.TILE_256x128, ds.TILE_128x256])
def test_gated_slices(tile):
    # gate and up columns of a slice are multiplied after the sums; ragged rows, slices of odd numbers of them
    for M, ksplit in ((100, 2), (100, 8), (131, 3), (9, 6)):
        t = inputs.swiglu(M, 1536, 384, 264, seed=M)
        Href, Yref = oracle.swiglu_chain(inputs.to_f64(t["X"]), inputs.to_f64(t["Wgu"]), inputs.to_f64(t["W2"]))
        print(f"gated slices tile={tile} M={M} ksplit={ksplit}", flush=True)
        pol = ds.SyncPolicy(ds.TILESYNC, ksplit=ksplit)
        res = [run_gemm_chain(t["X"], t["Wgu"], t["W2"], pol, mode, mid=ds.MID_SWIGLU, tile=tile) for mode in MODES]
        for H, Y in res:
            # (two roundings of products as heavy-tailed as these: the bounds of the other gated chains)
            assert mid_err(H, Href) <= TOL_MID and mid_err(Y, Yref) <= 1e-2
            assert torch.equal(H, res[0][0]) and torch.equal(Y, res[0][1])
        assert pol.status().timed_out == 0
        pol.destroy()


@pytest.mark.parametrize("tile", SLICED)
@pytest.mark.parametrize("mid,act,dtype", [(ds.MID_GELU, oracle.ACT_GELU, torch.float16), (ds.MID_RELU, oracle.ACT_RELU, torch.bfloat16)])
def test_activations_of_slices_and_packed_weights(tile, mid, act, dtype):
    for M, ksplit in ((5, 3), (66, 8), (133, 2)):
        t = inputs.mlp(M, 1536, 768, 264, seed=M, dtype=dtype)
        Href, Yref = oracle.gemm_chain(inputs.to_f64(t["X"]), inputs.to_f64(t["W1"]), inputs.to_f64(t["W2"]), act)
        print(f"slices of activations tile={tile} M={M} ksplit={ksplit} mid={mid}", flush=True)
        pol = ds.SyncPolicy(ds.ROWSYNC, ksplit=ksplit)
        res = [run_gemm_chain(t["X"], t["W1"], t["W2"], pol, mode, mid=mid, tile=tile) for mode in MODES]
        X, W1t, W2t = t["X"].cuda(), t["W1"].t().contiguous().cuda(), t["W2"].t().contiguous().cuda()
        Hp, Yp = (torch.full((M, n), float("nan"), dtype=dtype, device="cuda") for n in (768, 264))
        ds.dep_gemm_chain(X, ds.pack_weights_kblocked(W1t), Hp, ds.pack_weights_kblocked(W2t), Yp, pol, mode=ds.MODE_FUSED, mid=mid, tile=tile)
        torch.cuda.synchronize()
        for H, Y in res + [(Hp, Yp)]:
            if dtype == torch.float16:
                assert rel_err(H, Href) <= TOL_FP16 and rel_err(Y, Yref) <= TOL_FP16
            else:
                assert mid_err(H, Href) <= TOL_MID and rel_err(Y, Yref) <= TOL_BF16
            assert torch.equal(H, res[0][0]) and torch.equal(Y, res[0][1])
        assert pol.status().timed_out == 0
        pol.destroy()


@pytest.mark.parametrize("tile", SLICED)
@pytest.mark.parametrize("kind", [ds.ROWSYNC, ds.TILESYNC, ds.STRIDEDSYNC])
def test_slices_of_a_middle_convolution(tile, kind):
    # the middle stage waits, exchanges slices and posts; 128 channels are 18 K steps, in three parts of whole filter rows
    t = [inputs.conv(2, 9, 11, c, 128 if c == 64 else 192, 64, seed=c) for c in (64, 128)] + [inputs.conv(2, 9, 11, 192, 72, 64, seed=3)]
    x, ws = t[0]["x"], [a["w1"] for a in t]
    xd, wd = x.cuda(), [w.cuda() for w in ws]
    pol = ds.SyncPolicy(kind, ksplit=3)
    res = []
    for mode in MODES:
        print(f"slices of convolutions tile={tile} kind={kind} mode={mode}", flush=True)
        outs = [torch.full((2, 9, 11, w.shape[0]), float("nan"), dtype=x.dtype, device="cuda") for w in ws]
        ds.dep_conv_chain_n(xd, wd, outs, pol, mode=mode, tile=tile)
        torch.cuda.synchronize()
        res.append(outs)
    info = ds.conv_chain_n_plan(xd, wd, res[0], pol, tile=tile)
    assert info.n_mid == 3 * info.mid_grid_x * info.mid_grid_y
    for outs in res:
        assert all(torch.equal(a, b) for a, b in zip(outs, res[0]))
    for i in range(3):                                     # each stage against the oracle on the input that it really read
        prev = inputs.to_f64(x) if i == 0 else res[0][i - 1].cpu().double().numpy()
        ref = oracle.conv2d_nhwc(prev, inputs.to_f64(ws[i]), oracle.ACT_NONE if i == 2 else oracle.ACT_RELU)
        assert (rel_err(res[0][i], ref) <= TOL_BF16) if i == 2 else (mid_err(res[0][i], ref) <= TOL_MID), i
    assert pol.status().timed_out == 0
    pol.destroy()


@pytest.mark.parametrize("M,K1,N1,N2", [(16, 5312, 1088, 264), (1, 6592, 1856, 72), (100, 4544, 832, 200), (300, 4288, 1472, 520)])
def test_parts_that_differ_by_a_piece(M, K1, N1, N2):
    # numbers of K steps that the library's own split does not divide (83, 103, 71 and 67 in the first stage)
    ops, H, Y = whole_numbers(M, K1, N1, N2)
    uneven = 0
    for tile in [ds.TILE_AUTO, ds.TILE_64x64] + SLICED:
        print(f"uneven parts M={M} K1={K1} tile={tile}", flush=True)
        for kind in (ds.ROWSYNC, ds.TILESYNC):
            pol = ds.SyncPolicy(kind)
            for mode in MODES:
                h, y = run_gemm_chain(*ops, pol, mode, mid=ds.MID_NONE, tile=tile)
                assert torch.equal(h.cpu().float(), H) and torch.equal(y.cpu(), Y)
            assert pol.status().timed_out == 0
            a = [t.cuda().contiguous() for t in (ops[0], ops[1].t(), ops[2].t())]
            plan = ds.gemm_chain_plan(a[0], a[1], torch.empty_like(h), a[2], torch.empty_like(y), pol, mid=ds.MID_NONE, tile=tile)
            uneven += (K1 // 64) % (plan.n_prod // (plan.prod_grid_x * plan.prod_grid_y)) != 0
            pol.destroy()
    assert uneven >= 6


@pytest.mark.parametrize("tile", [ds.TILE_AUTO, ds.TILE_64x64] + SLICED + [ds.TILE_192x192])
def test_unequal_parts_of_strided_and_gated_chains(tile):
    # StridedSync (semaphores shared by every third column tile) and the gated product, with parts that differ; an activation on the way
    print(f"uneven parts, strided and gated, tile={tile}", flush=True)
    for M, K1, N1, N2, mid in ((40, 5312, 1152, 264, ds.MID_GELU), (90, 4544, 1472, 200, ds.MID_SWIGLU)):
        if mid == ds.MID_SWIGLU and tile in (ds.TILE_64x64, ds.TILE_64x192, ds.TILE_128x192_DEEP, ds.TILE_192x192):
            continue                                      # (no gate and up pairs in a wave)
        t = (inputs.swiglu if mid == ds.MID_SWIGLU else inputs.mlp)(M, K1, N1, N2, seed=M)
        W1 = t["Wgu" if mid == ds.MID_SWIGLU else "W1"]
        args = [inputs.to_f64(x) for x in (t["X"], W1, t["W2"])]
        Href, Yref = oracle.swiglu_chain(*args) if mid == ds.MID_SWIGLU else oracle.gemm_chain(*args, oracle.ACT_GELU)
        for kind in (ds.STRIDEDSYNC, ds.TILESYNC):
            pol = ds.SyncPolicy(kind, count=1)
            res = [run_gemm_chain(t["X"], W1, t["W2"], pol, mode, mid=mid, tile=tile) for mode in MODES]
            assert pol.status().timed_out == 0
            a = [x.cuda().contiguous() for x in (t["X"], W1.t(), t["W2"].t())]
            plan = ds.gemm_chain_plan(a[0], a[1], torch.empty_like(res[0][0]), a[2], torch.empty_like(res[0][1]), pol, mid=mid, tile=tile)
            assert (K1 // 64) % (plan.n_prod // (plan.prod_grid_x * plan.prod_grid_y))
            pol.destroy()
            assert mid_err(res[0][0], Href) <= TOL_MID and rel_err(res[0][1], Yref) <= TOL_BF16
            for other in res[1:]:
                assert all(torch.equal(x, y) for x, y in zip(res[0], other))
