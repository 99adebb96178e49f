"""Chains whose tiles are all resident at once, which the library runs with 64x64 tiles of which three share a
CU: sizes around the 32-row blocks and the tile, splits that divide and that do not, every launch mode."""
import pytest
import torch

import inputs
import oracle
import paper_2305_13450_amd as ds
from gpu_util import TOL_BF16, TOL_MID, mid_err, rel_err, run_conv_chain, run_gemm_chain

pytestmark = pytest.mark.gpu

MODES = [ds.MODE_FUSED, ds.MODE_FINE, ds.MODE_STREAMSYNC, ds.MODE_PLAIN]


@pytest.mark.parametrize("split", [0, 1, 3, 8])
@pytest.mark.parametrize("M", [1, 8, 9, 31, 33, 64, 65, 129])
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

