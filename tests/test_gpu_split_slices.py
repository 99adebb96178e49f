"""Tiles split along K of which every part finishes a slice of the rows: slices of odd and no rows, every number of
parts, and parts that end before others of their tile have been started.  Inputs are small whole numbers whose
sums are exact in fp32 and in bf16, so every result is compared bit for bit."""
import pytest
import torch

import paper_2305_13450_amd as ds
from gpu_util import run_gemm_chain

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
    for flags, modes in ((0, MODES), (ds.FLAG_HW_ORDER, [ds.MODE_STREAMSYNC, ds.MODE_FUSED])):
        pol = ds.SyncPolicy(ds.ROWSYNC, ksplit=8, flags=flags)
        for mode in modes:
            for _ in range(2):
                h, y = run_gemm_chain(*ops, pol, mode, mid=ds.MID_NONE, tile=tile)
                assert torch.equal(h.cpu().float(), H) and torch.equal(y.cpu(), Y)
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
