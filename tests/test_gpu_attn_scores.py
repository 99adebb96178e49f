"""The prompt-phase attention tile where its running reference matters: scores that grow along the
sequence (a new maximum in most key blocks), scores that differ by hundreds (one key carries a row),
and equal ones, over sequence ends and cache ends that cut a block of 64 keys anywhere."""
import pytest
import torch

import inputs
import oracle
import paper_2305_13450_amd as ds
from gpu_util import TOL_BF16, row_err, run_attn_chain

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
# deviations: 2e-2 covers both.
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
        assert row_err(T, ref) <= TOL_BF16
