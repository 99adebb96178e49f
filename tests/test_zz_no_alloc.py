"""GPU test of the allocation-free entry point dep_gemm_chain_static: through the C ABI, its output
must be bit-identical to dep_gemm_chain's (one dispatch, same policy kind and parameters), on calls
in a row that share the library's static device workspace, the later ones smaller than the first."""
import ctypes

import pytest
import torch

import inputs
import paper_2305_13450_amd as ds
from gpu_util import same

pytestmark = pytest.mark.gpu


def _chain(t, mid):
    X = t["X"].cuda()
    W1 = t["Wgu" if mid == ds.MID_SWIGLU else "W1"]
    W1t, W2t = W1.t().contiguous().cuda(), t["W2"].t().contiguous().cuda()
    n1 = W1.shape[1] // 2 if mid == ds.MID_SWIGLU else W1.shape[1]
    return X, W1t, W2t, n1


def _outputs(M, n1, n2, dtype):
    return (torch.full((M, n1), float("nan"), dtype=dtype, device="cuda"),
            torch.full((M, n2), float("nan"), dtype=dtype, device="cuda"))


def _both(t, mid, kind, stream=None, **params):
    """(H, Y) of the static entry point and of dep_gemm_chain in one-dispatch mode."""
    X, W1t, W2t, n1 = _chain(t, mid)
    M, n2 = X.shape[0], W2t.shape[0]
    Hs, Ys = _outputs(M, n1, n2, X.dtype)
    torch.cuda.synchronize()
    ds.dep_gemm_chain_static(X, W1t, Hs, W2t, Ys, kind, mid=mid, stream=stream, **params)
    torch.cuda.synchronize()
    pol = ds.SyncPolicy(kind, **params)
    H, Y = _outputs(M, n1, n2, X.dtype)
    torch.cuda.synchronize()
    ds.dep_gemm_chain(X, W1t, H, W2t, Y, pol, mode=ds.MODE_FUSED, mid=mid, stream_producer=stream)
    torch.cuda.synchronize()
    assert pol.status().timed_out == 0
    pol.destroy()
    return (Hs, Ys), (H, Y)


def test_static_entry_matches_the_allocating_one_on_calls_in_a_row():
    print("static entry: 640 rows (split along K), then 200 rows, then 1 row, then 640 again", flush=True)
    # the first chain is split along K (few tiles on 256 CUs), so it uses semaphores, arrival
    # counters and partial tiles of the static array; the following, smaller ones find all of
    # that as the first left it
    big = inputs.mlp(640, 4096, 1536, 1024, seed=5)
    small = inputs.mlp(200, 512, 768, 320, seed=6)
    one = inputs.mlp(1, 4096, 1536, 1024, seed=7)
    for t, kind in ((big, ds.ROWSYNC), (small, ds.TILESYNC), (one, ds.ROWSYNC), (big, ds.TILESYNC), (small, ds.TILESYNC)):
        (Hs, Ys), (H, Y) = _both(t, ds.MID_GELU, kind)
        assert not torch.isnan(Ys).any()
        assert same(Hs, H, "H static/policy") and same(Ys, Y, "Y static/policy")


def test_static_entry_gated_mlp_and_side_stream():
    t = inputs.swiglu(300, 1024, 1408, 512, seed=8)
    s = torch.cuda.Stream()
    for kind in (ds.TILESYNC, ds.STRIDEDSYNC, ds.ROWSYNC):
        (Hs, Ys), (H, Y) = _both(t, ds.MID_SWIGLU, kind, stream=s, count=2 if kind == ds.STRIDEDSYNC else 0)
        assert same(Hs, H, "H static/policy") and same(Ys, Y, "Y static/policy")
    # repeated chains of one geometry back to back without a host synchronisation in between
    X, W1t, W2t, n1 = _chain(t, ds.MID_SWIGLU)
    outs = [_outputs(300, n1, 512, X.dtype) for _ in range(6)]
    torch.cuda.synchronize()
    for Hs, Ys in outs:
        ds.dep_gemm_chain_static(X, W1t, Hs, W2t, Ys, ds.TILESYNC, mid=ds.MID_SWIGLU, stream=s)
    torch.cuda.synchronize()
    for Hs, Ys in outs[1:]:
        assert same(Hs, outs[0][0]) and same(Ys, outs[0][1])


def test_static_entry_rejects_what_does_not_fit():
    # 32768 producer tiles under TileSync need more semaphores than the static workspace holds
    M, K1, N1, N2 = 8192, 64, 16384, 64
    X = torch.zeros((M, K1), dtype=torch.bfloat16, device="cuda")
    W1t = torch.zeros((N1, K1), dtype=torch.bfloat16, device="cuda")
    W2t = torch.zeros((N2, N1), dtype=torch.bfloat16, device="cuda")
    H = torch.zeros((M, N1), dtype=torch.bfloat16, device="cuda")
    Y = torch.full((M, N2), 7.0, dtype=torch.bfloat16, device="cuda")
    with pytest.raises(ds.DepsyncError) as e:
        ds.dep_gemm_chain_static(X, W1t, H, W2t, Y, ds.TILESYNC, tile=ds.TILE_64x64)
    assert e.value.status == ds.ELIMIT
    with pytest.raises(ds.DepsyncError) as e:      # no trace area
        ds.dep_gemm_chain_static(X, W1t, H, W2t, Y, ds.ROWSYNC, flags=ds.FLAG_TRACE)
    assert e.value.status == ds.EINVAL
    d = ds._gemm_desc(X, W1t, H, W2t, Y, ds.MID_GELU, ds.TILE_AUTO)
    assert ds._lib().dep_gemm_chain_static(ctypes.byref(d), 9, None, None) == ds.EINVAL
    assert ds._lib().dep_gemm_chain_static(None, ds.ROWSYNC, None, None) == ds.EINVAL
    torch.cuda.synchronize()
    assert bool((Y == 7.0).all())                  # nothing was enqueued


def test_static_entry_takes_a_split_that_fits_with_another_shape():
    # the caller's eight parts (six and three here) of the library's 256x128 tiles need more scratch than there is, of 64x128 tiles not
    t = inputs.swiglu(192, 384, 12480, 6664, seed=9)
    X, W1t, W2t, n1 = _chain(t, ds.MID_SWIGLU)
    (H0, Y0), (Hs, Ys), (H, Y) = (_outputs(192, n1, 6664, X.dtype) for _ in range(3))
    print("static entry: forced split near the end of the scratch", flush=True)
    pol = ds.SyncPolicy(ds.ROWSYNC, ksplit=8)
    info = ds.gemm_chain_plan(X, W1t, H, W2t, Y, pol, mid=ds.MID_SWIGLU)
    rows, cols = ds.tile_shape(info.tile_prod)
    assert (info.n_prod + info.n_cons) * rows * cols > 32 << 20
    with pytest.raises(ds.DepsyncError) as e:
        ds.dep_gemm_chain_static(X, W1t, H0, W2t, Y0, ds.ROWSYNC, mid=ds.MID_SWIGLU, ksplit=8, tile=info.tile_prod)
    assert e.value.status == ds.ELIMIT
    ds.dep_gemm_chain_static(X, W1t, Hs, W2t, Ys, ds.ROWSYNC, mid=ds.MID_SWIGLU, ksplit=8)
    ds.dep_gemm_chain(X, W1t, H, W2t, Y, pol, mode=ds.MODE_FUSED, mid=ds.MID_SWIGLU, tile=ds.TILE_64x128)
    torch.cuda.synchronize()
    assert pol.status().timed_out == 0 and same(Hs, H, "H") and same(Ys, Y, "Y")
    pol.destroy()


def test_a_policy_takes_a_split_that_fits_with_another_shape():
    # 41449 tiles of 256x128 have no arrival counter each in a policy's workspace (32768), 27709 of 256x192 do
    X = torch.empty((64, 64), dtype=torch.bfloat16, device="cuda")        # (planned only)
    d = ds._gemm_desc(X, X, X, X, X, ds.MID_NONE, ds.TILE_AUTO)
    d.M, d.K1, d.N1, d.N2 = 58453, 512, 23104, 72
    d.ldx = d.ldw1 = 512
    d.ldh = d.ldw2 = 23104
    d.ldy = 72
    info = ds.PlanInfo()
    for ksplit, tile in ((1, ds.TILE_256x128), (2, ds.TILE_256x192)):
        pol = ds.SyncPolicy(ds.ROWSYNC, ksplit=ksplit)
        assert ds._lib().depsync_gemm_chain_plan(ctypes.byref(d), pol.handle, 0, ctypes.byref(info)) == ds.OK
        assert info.tile_prod == tile
        pol.destroy()


def test_a_chain_that_needs_scratch_is_captured_by_a_policy_without():
    # the library's choice splits the second convolution; under capture there is no scratch to allocate, and the former shape needs none
    g = torch.Generator().manual_seed(4)
    x = torch.randn((2, 131, 25, 64), generator=g).to(torch.bfloat16).cuda()
    ws = [(torch.randn((k, 3, 3, c), generator=g) * (2 / (9 * c)) ** 0.5).to(torch.bfloat16).cuda() for c, k in ((64, 704), (704, 392))]
    outs = [[torch.zeros((2, 131, 25, k), dtype=torch.bfloat16, device="cuda") for k in (704, 392)] for _ in range(2)]
    warm, cold = ds.SyncPolicy(ds.STRIDEDSYNC), ds.SyncPolicy(ds.STRIDEDSYNC)
    info = ds.conv_chain_plan(x, ws[0], outs[0][0], ws[1], outs[0][1], warm)
    assert info.n_cons == 3 * info.cons_grid_x * info.cons_grid_y
    print("capture without scratch", flush=True)
    ds.dep_conv_chain(x, ws[0], outs[0][0], ws[1], outs[0][1], warm, mode=ds.MODE_STREAMSYNC, tile=ds.TILE_64x128)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        ds.dep_conv_chain(x, ws[0], outs[1][0], ws[1], outs[1][1], cold, mode=ds.MODE_FUSED, stream_producer=torch.cuda.current_stream())
    graph.replay()
    torch.cuda.synchronize()
    assert cold.status().timed_out == 0
    assert same(outs[1][0], outs[0][0], "mid") and same(outs[1][1], outs[0][1], "out")
    del graph
    warm.destroy()
    cold.destroy()


def test_a_split_asked_for_runs_with_a_shape_that_fits():
    # two parts of the shape that the library chooses for the first chain are more than the fixed workspace holds, and the second chain's
    # would need scratch in a capture: other shapes leave less, or have no two parts that start on a producer tile
    for M, K1, N1, N2, kind in ((2669, 2944, 6016, 24, ds.ROWSYNC), (4556, 576, 1920, 24, ds.TILESYNC)):
        t = inputs.mlp(M, K1, N1, N2, seed=M)
        X, W1t, W2t, n1 = _chain(t, ds.MID_NONE)
        H, Y = _outputs(M, n1, N2, X.dtype)
        print(f"a split asked for, M={M}", flush=True)
        if kind == ds.ROWSYNC:
            ds.dep_gemm_chain_static(X, W1t, H, W2t, Y, kind, mid=ds.MID_NONE, ksplit=2)
        else:
            pol = ds.SyncPolicy(kind, ksplit=2)
            graph = torch.cuda.CUDAGraph()
            with torch.cuda.graph(graph):
                ds.dep_gemm_chain(X, W1t, H, W2t, Y, pol, mode=ds.MODE_FUSED, mid=ds.MID_NONE, stream_producer=torch.cuda.current_stream())
            graph.replay()
        torch.cuda.synchronize()
        Href = X.double() @ W1t.double().t()
        for got, ref in ((H, Href), (Y, Href @ W2t.double().t())):
            assert float((got.double() - ref).norm() / ref.norm()) <= 1e-2
    assert pol.status().timed_out == 0
    del graph
    pol.destroy()


@pytest.mark.parametrize("M,K1,N1,N2,kind", [(597, 2432, 4544, 1376, ds.TILESYNC), (138, 640, 5568, 12816, ds.ROWSYNC),
                                             (244, 3392, 11264, 14312, ds.ROWSYNC)])
def test_a_chain_that_every_choice_splits_is_captured_by_a_policy_without_scratch(M, K1, N1, N2, kind):
    # the library's choice and the former one split these (their tiles do not fill the chip); whole tiles need no scratch
    t = inputs.mlp(M, K1, N1, N2, seed=M)
    X, W1t, W2t, n1 = _chain(t, ds.MID_GELU)
    H, Y = _outputs(M, n1, N2, X.dtype)
    pol = ds.SyncPolicy(kind)
    print(f"capture without scratch M={M}", flush=True)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        ds.dep_gemm_chain(X, W1t, H, W2t, Y, pol, mode=ds.MODE_FUSED, stream_producer=torch.cuda.current_stream())
    Href = torch.nn.functional.gelu(X.double() @ W1t.double().t())
    Yref = Href @ W2t.double().t()
    for _ in range(3):
        H.fill_(float("nan")); Y.fill_(float("nan"))
        graph.replay()
        torch.cuda.synchronize()
        for got, ref in ((H, Href), (Y, Yref)):
            assert float((got.double() - ref).norm() / ref.norm()) <= 1e-2    # (bf16: 2.4e-3 by its roundings alone)
    assert pol.status().timed_out == 0
    del graph
    pol.destroy()


def _replays(graph, poison, results, want, between):
    for it in range(4):
        for t in poison:
            t.fill_(float("nan"))
        graph.replay()
        torch.cuda.synchronize()
        for got, ref in zip(results, want):
            assert same(got, ref, f"replay {it}")
        between(it)
        torch.cuda.synchronize()


@pytest.mark.parametrize("M,K1,N1,N2", [(64, 1024, 1536, 512), (640, 4096, 1536, 1024), (2048, 256, 6144, 1024)])
@pytest.mark.parametrize("kind", [ds.ROWSYNC, ds.TILESYNC])
def test_captured_chains_give_the_same_on_every_replay(M, K1, N1, N2, kind):
    # resident at once, split along K, and drawn from the queues; the workspace is used by other chains between the replays
    t, other = inputs.mlp(M, K1, N1, N2, seed=11), inputs.mlp(200, 512, 768, 320, seed=12)
    X, W1t, W2t, n1 = _chain(t, ds.MID_GELU)
    Xo, W1o, W2o, no = _chain(other, ds.MID_GELU)
    (H, Y), (Hs, Ys), (Hp, Yp) = (_outputs(M, n1, N2, X.dtype) for _ in range(3))
    (Ho, Yo), (Ho1, Yo1) = (_outputs(200, no, 320, X.dtype) for _ in range(2))
    pol, ref = ds.SyncPolicy(kind), ds.SyncPolicy(kind)
    print(f"capture and replay {M}x{K1}x{N1}x{N2} kind={kind}", flush=True)
    ds.dep_gemm_chain(X, W1t, H, W2t, Y, ref, mode=ds.MODE_STREAMSYNC)
    ds.dep_gemm_chain(Xo, W1o, Ho, W2o, Yo, ref, mode=ds.MODE_STREAMSYNC)
    ds.dep_gemm_chain(X, W1t, Hp, W2t, Yp, pol, mode=ds.MODE_FUSED)        # (scratch is allocated here)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        st = torch.cuda.current_stream()
        ds.dep_gemm_chain_static(X, W1t, Hs, W2t, Ys, kind, stream=st)
        ds.dep_gemm_chain(X, W1t, Hp, W2t, Yp, pol, mode=ds.MODE_FUSED, stream_producer=st)

    def between(it):
        # the other chain, and the captured one without the graph
        for x, w1, h, w2, y in ((Xo, W1o, Ho1, W2o, Yo1), (X, W1t, Hp, W2t, Yp), (X, W1t, Hp, W2t, Yp))[it % 2:]:
            for out in (h, y):
                out.fill_(float("nan"))
            ds.dep_gemm_chain_static(x, w1, h, w2, y, kind)
            torch.cuda.synchronize()
            assert same(h, Ho if x is Xo else H) and same(y, Yo if x is Xo else Y)
            for out in (h, y):
                out.fill_(float("nan"))
            ds.dep_gemm_chain(x, w1, h, w2, y, pol, mode=ds.MODE_FINE if it & 2 else ds.MODE_FUSED)
            torch.cuda.synchronize()
            assert same(h, Ho if x is Xo else H) and same(y, Yo if x is Xo else Y)
    _replays(graph, (Hs, Ys, Hp, Yp), (Hs, Ys, Hp, Yp), (H, Y, H, Y), between)
    assert pol.status().timed_out == 0
    del graph
    pol.destroy()
    ref.destroy()


@pytest.mark.parametrize("mode", [ds.MODE_FUSED, ds.MODE_FINE])
def test_a_chain_captured_after_side_launches(mode):
    # 1024 producer tiles on 512 slots: the two-stream form has side launches, which a capture and its replays must not meet
    M, K1, N1, N2 = 4096, 128, 1024, 256
    t = inputs.mlp(M, K1, N1, N2, seed=1)
    X, W1t, W2t, n1 = _chain(t, ds.MID_GELU)
    (H, Y), (Hp, Yp) = (_outputs(M, n1, N2, X.dtype) for _ in range(2))
    pol = ds.SyncPolicy(ds.ROWSYNC)
    assert ds.launch_form(ds._gemm_desc(X, W1t, H, W2t, Y, ds.MID_GELU, ds.TILE_64x64), pol, ds.MODE_FINE) == (2, False)
    print(f"capture after side launches mode={mode}", flush=True)
    ds.dep_gemm_chain(X, W1t, H, W2t, Y, pol, mode=ds.MODE_FINE, tile=ds.TILE_64x64)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        ds.dep_gemm_chain(X, W1t, Hp, W2t, Yp, pol, mode=mode, tile=ds.TILE_64x64, stream_producer=torch.cuda.current_stream())

    def between(it):
        Y.fill_(float("nan"))
        ds.dep_gemm_chain(X, W1t, H, W2t, Y, pol, mode=ds.MODE_FINE, tile=ds.TILE_64x64)
        graph.replay()                                                     # right behind, no host sync in between
    want = (H.clone(), Y.clone())
    _replays(graph, (Hp, Yp), (Hp, Yp, H, Y), want * 2, between)
    assert pol.status().timed_out == 0
    del graph
    pol.destroy()


def test_a_captured_chain_keeps_its_scratch_when_a_larger_chain_follows():
    # both are split along K; the second needs more scratch than the policy has after the first, whose graph goes on using its own
    t, big = inputs.mlp(64, 4096, 1536, 1024, seed=21), inputs.mlp(640, 4096, 1536, 1024, seed=22)
    X, W1t, W2t, n1 = _chain(t, ds.MID_GELU)
    Xb, W1b, W2b, nb = _chain(big, ds.MID_GELU)
    (H, Y), (Hw, Yw) = (_outputs(64, n1, 1024, X.dtype) for _ in range(2))
    (Hb, Yb), (Hc, Yc) = (_outputs(640, nb, 1024, X.dtype) for _ in range(2))
    pol, fresh = ds.SyncPolicy(ds.ROWSYNC), ds.SyncPolicy(ds.ROWSYNC)
    small, large = (ds.gemm_chain_plan(x, a, h, b, y, pol) for x, a, h, b, y in ((X, W1t, H, W2t, Y), (Xb, W1b, Hb, W2b, Yb)))
    parts = [(i.n_prod, i.n_cons, i.prod_grid_x * i.prod_grid_y, i.cons_grid_x * i.cons_grid_y) for i in (small, large)]
    assert all(p[0] > p[2] or p[1] > p[3] for p in parts), parts
    print("a captured chain, then a larger one", flush=True)
    ds.dep_gemm_chain(X, W1t, Hw, W2t, Yw, pol, mode=ds.MODE_FUSED)                   # the scratch that the capture finds
    ds.dep_gemm_chain(Xb, W1b, Hc, W2b, Yc, fresh, mode=ds.MODE_FUSED)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        ds.dep_gemm_chain(X, W1t, H, W2t, Y, pol, mode=ds.MODE_FUSED, stream_producer=torch.cuda.current_stream())

    def between(_):
        ds.dep_gemm_chain(Xb, W1b, Hb, W2b, Yb, pol, mode=ds.MODE_FUSED)
        torch.cuda.synchronize()
        assert same(Hb, Hc, "H of the larger") and same(Yb, Yc, "Y of the larger")

    between(0)
    _replays(graph, (H, Y), (H, Y), (Hw, Yw), between)
    assert pol.status().timed_out == 0
    del graph
    pol.destroy()
    fresh.destroy()
