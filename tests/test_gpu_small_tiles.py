"""Chains whose tiles are all resident at once, which the library runs with 64x64 tiles of which three share a
CU: sizes around the 32-row blocks and the tile, splits that divide and that do not, every launch mode."""
import pytest
import torch

import inputs
import oracle
import paper_2305_13450_amd as ds
from gpu_util import TOL_BF16, TOL_FP16, TOL_MID, mid_err, rel_err, row_err, run_conv_chain, run_gemm_chain

pytestmark = pytest.mark.gpu

MODES = [ds.MODE_FUSED, ds.MODE_FINE, ds.MODE_STREAMSYNC, ds.MODE_PLAIN]


@pytest.mark.parametrize("split", [0, 1, 3, 8])
@pytest.mark.parametrize("M", [1, 8, 9, 31, 32, 33, 64, 65, 129])
def test_rows_and_splits(M, split):
    K1, N1, N2 = 1536, 192, 200
    t = inputs.mlp(M, K1, N1, N2, seed=M)
    print(f"small tiles M={M} split={split}", flush=True)
    Href, Yref = oracle.gemm_chain(inputs.to_f64(t["X"]), inputs.to_f64(t["W1"]), inputs.to_f64(t["W2"]), oracle.ACT_GELU)
    for kind in (ds.TILESYNC, ds.ROWSYNC):
        pol = ds.SyncPolicy(kind, ksplit=split)
        res = [run_gemm_chain(t["X"], t["W1"], t["W2"], pol, mode) for mode in MODES]
        assert pol.status().timed_out == 0
        pol.destroy()
        assert mid_err(res[0][0], Href) <= TOL_MID
        assert rel_err(res[0][1], Yref) <= TOL_BF16
        for other in res[1:]:
            assert all(torch.equal(a, b) for a, b in zip(res[0], other))


@pytest.mark.parametrize("kind", [ds.ROWSYNC, ds.TILESYNC, ds.STRIDEDSYNC])
@pytest.mark.parametrize("B,H,W", [(1, 7, 9), (2, 13, 11)])
def test_convolutions(B, H, W, kind):
    t = inputs.conv(B, H, W, 128, 128, 72, seed=3)
    print(f"small tiles conv {B}x{H}x{W} kind={kind}", flush=True)
    mid_ref, ref = oracle.conv_chain(inputs.to_f64(t["x"]), inputs.to_f64(t["w1"]), inputs.to_f64(t["w2"]))
    for split in (0, 1, 3):
        pol = ds.SyncPolicy(kind, ksplit=split)
        res = [run_conv_chain(t["x"], t["w1"], t["w2"], pol, mode) for mode in MODES]
        assert pol.status().timed_out == 0
        pol.destroy()
        assert mid_err(res[0][0], mid_ref) <= TOL_MID
        assert rel_err(res[0][1], ref) <= TOL_BF16
        for other in res[1:]:
            assert all(torch.equal(a, b) for a, b in zip(res[0], other))



@pytest.mark.parametrize("mid,act", [(ds.MID_NONE, oracle.ACT_NONE), (ds.MID_RELU, oracle.ACT_RELU), (ds.MID_GELU, oracle.ACT_GELU)])
@pytest.mark.parametrize("M", [1, 65, 130])
def test_fp16_and_the_other_middles(M, mid, act):
    t = inputs.mlp(M, 1024, 320, 136, seed=M, dtype=torch.float16)
    print(f"small tiles fp16 M={M} mid={mid}", flush=True)
    Href, Yref = oracle.gemm_chain(inputs.to_f64(t["X"]), inputs.to_f64(t["W1"]), inputs.to_f64(t["W2"]), act)
    for kind in (ds.TILESYNC, ds.ROWSYNC):
        pol = ds.SyncPolicy(kind)
        res = [run_gemm_chain(t["X"], t["W1"], t["W2"], pol, mode, mid=mid) for mode in MODES]
        assert pol.status().timed_out == 0
        pol.destroy()
        # an intermediate may be off by its own rounding (2^-11) and as much again
        assert mid_err(res[0][0], Href, ulp=2.0 ** -10) <= TOL_MID and rel_err(res[0][1], Yref) <= TOL_FP16
        for other in res[1:]:
            assert all(torch.equal(a, b) for a, b in zip(res[0], other))


# keys of a (head, sequence) pair: too few for a second part, one more part than fits a third of the slots
# otherwise, and the most parts a pair can have
@pytest.mark.parametrize("dtype,tol", [(torch.bfloat16, TOL_BF16), (torch.float16, TOL_FP16)])
@pytest.mark.parametrize("batch,cached,heads", [(1, 300, 2), (5, 511, 13), (4, 1000, 16), (1, 2600, 3)])
def test_token_generation(batch, cached, heads, dtype, tol):
    E, K1, N2 = heads * 128, 512, 200
    t = inputs.attention(batch, K1, heads, 128, N2, seed=heads, dtype=dtype)
    kv = inputs.kv_cache(batch, cached, heads, 128, seed=cached, dtype=dtype)
    X, Wq, Wo = t["X"].cuda(), t["Wqkv"].t().contiguous().cuda(), t["Wo"].t().contiguous().cuda()
    Kc, Vc = kv["Kc"].cuda(), kv["Vc"].cuda()
    kw = dict(mid=ds.MID_CAUSAL_ATTN, batch=batch, seq=1, heads=heads, head_dim=128, k_cache=Kc, v_cache=Vc)
    print(f"small tiles generation {batch}x{cached} heads={heads} {dtype}", flush=True)
    for kind in (ds.STRIDEDSYNC, ds.ROWSYNC):
        pol = ds.SyncPolicy(kind)
        res = []
        for mode in MODES:
            QKV, T, Y = (torch.full((batch, n), float("nan"), dtype=dtype, device="cuda") for n in (3 * E, E, N2))
            assert ds.gemm_chain_plan(X, Wq, QKV, Wo, Y, pol, T=T, **kw).slots == 3 * ds.device_info()[0]
            ds.dep_gemm_chain(X, Wq, QKV, Wo, Y, pol, mode=mode, T=T, **kw)
            torch.cuda.synchronize()
            res.append((QKV, T, Y))
        assert pol.status().timed_out == 0
        pol.destroy()
        QKV, T, Y = res[0]
        assert row_err(T, oracle.cached_attention(inputs.to_f64(QKV.cpu()), inputs.to_f64(kv["Kc"]), inputs.to_f64(kv["Vc"]), batch, 1, heads, 128)) <= tol
        assert rel_err(Y, oracle.gemm(inputs.to_f64(T.cpu()), inputs.to_f64(t["Wo"]))) <= tol
        for other in res[1:]:
            assert all(torch.equal(a, b) for a, b in zip(res[0], other))


# sizes for which the library takes 192x192 tiles under both kinds or the one named: part of a tile, a whole one, three with a ragged
# last one; whole and split stages (parts of 14 to 32 steps); a ragged last column tile of the producer, and 83 steps of the second stage
# in four parts of 21, 21, 21 and 20 (under TileSync, whose parts start on segments of three steps: of 21, 21, 21 and the rest)
@pytest.mark.parametrize("M,K1,N1,N2,dtype,kinds", [
    (129, 1088, 6144, 7000, torch.bfloat16, [ds.ROWSYNC]), (192, 1088, 6144, 7000, torch.float16, [ds.ROWSYNC]),
    (333, 2048, 6144, 6144, torch.bfloat16, [ds.ROWSYNC, ds.TILESYNC]), (570, 1536, 6144, 4000, torch.bfloat16, [ds.ROWSYNC, ds.TILESYNC]),
    (333, 2048, 5312, 6144, torch.bfloat16, [ds.ROWSYNC, ds.TILESYNC])])
def test_tiles_of_192_rows(M, K1, N1, N2, dtype, kinds):
    t = inputs.mlp(M, K1, N1, N2, seed=M, dtype=dtype)
    print(f"192 rows M={M}", flush=True)
    Href, Yref = oracle.gemm_chain(inputs.to_f64(t["X"]), inputs.to_f64(t["W1"]), inputs.to_f64(t["W2"]), oracle.ACT_GELU)
    for kind in kinds:
        pol = ds.SyncPolicy(kind)
        res = [run_gemm_chain(t["X"], t["W1"], t["W2"], pol, mode) for mode in MODES]
        a = [x.cuda().contiguous() for x in (t["X"], t["W1"].t(), t["W2"].t())]
        plan = ds.gemm_chain_plan(a[0], a[1], torch.empty_like(res[0][0]), a[2], torch.empty_like(res[0][1]), pol)
        assert plan.tile_prod == plan.tile_cons == ds.TILE_192x192
        assert (plan.prod_grid_x, plan.prod_grid_y) == (-(-N1 // 192), -(-M // 192))
        assert pol.status().timed_out == 0
        pol.destroy()
        assert mid_err(res[0][0], Href) <= TOL_MID
        assert rel_err(res[0][1], Yref) <= (TOL_BF16 if dtype == torch.bfloat16 else TOL_FP16)
        for other in res[1:]:
            assert all(torch.equal(a, b) for a, b in zip(res[0], other))


@pytest.mark.parametrize("packed", [False, True])
@pytest.mark.parametrize("M", [1, 5, 32])
def test_32_rows_with_packed_weights_padded_rows_and_uneven_parts(M, packed):
    # both stages in parts that differ by a step (83 and 47 steps, few tiles); rows of X and of the outputs further apart than they are long
    K1, N1, N2 = 5312, 3008, 328
    t = inputs.mlp(M, K1, N1, N2, seed=M)
    print(f"32 rows M={M} packed={packed}", flush=True)
    Href, Yref = oracle.gemm_chain(inputs.to_f64(t["X"]), inputs.to_f64(t["W1"]), inputs.to_f64(t["W2"]), oracle.ACT_RELU)
    W1t, W2t = (t[n].t().contiguous().cuda() for n in ("W1", "W2"))
    if packed:
        W1t, W2t = ds.pack_weights_kblocked(W1t), ds.pack_weights_kblocked(W2t)
    X = torch.zeros((M, K1 + 64), dtype=t["X"].dtype, device="cuda")[:, :K1]
    X.copy_(t["X"])
    for kind in (ds.ROWSYNC, ds.TILESYNC):
        pol = ds.SyncPolicy(kind)
        res = []
        for mode in MODES:
            H, Y = (torch.full((M, n + 64), float("nan"), dtype=X.dtype, device="cuda")[:, :n] for n in (N1, N2))
            plan = ds.gemm_chain_plan(X, W1t, H, W2t, Y, pol, mid=ds.MID_RELU)
            assert plan.slots == 3 * ds.device_info()[0] and plan.prod_grid_y == 1
            assert (K1 // 64) % (plan.n_prod // plan.prod_grid_x) and (N1 // 64) % (plan.n_cons // plan.cons_grid_x)
            ds.dep_gemm_chain(X, W1t, H, W2t, Y, pol, mode=mode, mid=ds.MID_RELU)
            torch.cuda.synchronize()
            res.append((H, Y))
        assert pol.status().timed_out == 0
        pol.destroy()
        assert mid_err(res[0][0], Href) <= TOL_MID and rel_err(res[0][1], Yref) <= TOL_BF16
        for other in res[1:]:
            assert all(torch.equal(a, b) for a, b in zip(res[0], other))


@pytest.mark.parametrize("mode", MODES)
def test_192x192_asked_for(mode):
    # ragged in rows and columns, the second stage unsplit, split by the library and by the caller
    t = inputs.mlp(333, 1280, 1728, 1000, seed=3)
    print(f"192x192 asked for, mode={mode}", flush=True)
    Href, Yref = oracle.gemm_chain(inputs.to_f64(t["X"]), inputs.to_f64(t["W1"]), inputs.to_f64(t["W2"]), oracle.ACT_GELU)
    for kind in (ds.ROWSYNC, ds.TILESYNC):
        for ksplit in (0, 1, 3):
            pol = ds.SyncPolicy(kind, ksplit=ksplit)
            H, Y = run_gemm_chain(t["X"], t["W1"], t["W2"], pol, mode, tile=ds.TILE_192x192)
            assert pol.status().timed_out == 0
            pol.destroy()
            assert mid_err(H, Href) <= TOL_MID and rel_err(Y, Yref) <= TOL_BF16
