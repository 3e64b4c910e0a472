"""GPU test of the ping-pong main loop (256 x 256, 320 x 256 and 256 x 128 tiles): forced on calls whose products have one K
step, two, and numbers around the ring's turn, with ragged last tiles and gathered rows in pieces of whole K steps
(64, 128) and not (96, 216), it gives bit for bit what the plain loop of the 128 x 128 tile gives -- an output
element is the same chain of matrix instructions in both.  (Without rotary embedding: which product of a rotary
pair is rounded before the sum depends on the tile's rows.)"""

import pytest
import torch

from oracle import vit_encode as O
from paper_2601_11590_amd import binding as B, workloads as W
from parity_util import check
from test_gpu_parity import case, parity, small

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("hidden,heads", [(64, 1), (128, 2), (192, 3), (256, 4), (320, 5), (96, 3), (216, 3)])
@pytest.mark.parametrize("merge", [1, 2, 4])
def test_large_tiles_give_the_bits_of_the_128_tile(hidden, heads, merge):
    cfg = small("bf16", hidden=hidden, num_heads=heads, head_dim=hidden // heads, rope="none", rope_pairs=(0, 0, 0), norm="layernorm",
                mlp_dim=2 * hidden + 72, out_dim=328, merge=merge)
    grids = [(1, 20, 32), (1, 4, 4), (1, 12, 8)]
    gw, layers, patches, cu, grid = case(cfg, grids)
    ref = O.encode(cfg, gw, layers, patches, cu, grid)
    enc = B.EpdEncoder(cfg, gw, layers, max_tokens=patches.shape[0], max_segments=len(grids), max_items=len(grids))
    p = B.to_device_patches(patches, cfg.dtype)
    out = {}
    for tile in (4, 0, 5, 2):
        enc.set_tuning(tile, 0)
        out[tile] = enc.encode(p, cu, grid).clone()
    torch.cuda.synchronize()
    check(cfg, out[0].float().cpu().numpy(), ref, "256 x 256")
    assert all(torch.equal(out[t], out[4]) for t in (0, 5, 2))
    enc.close()


@pytest.mark.parametrize("d,pairs", [(32, (0, 8, 8)), (64, (0, 16, 16)), (72, (0, 18, 18)), (80, (8, 16, 16)), (96, (16, 16, 16)), (128, (16, 24, 24))])
@pytest.mark.parametrize("tile", [0, 5, 2])
def test_rotary_table_of_every_head_dim(d, pairs, tile):
    """Tables of 8 to 32 chunks a token in LDS, swizzled and not, and those that do not fit (head_dim 128 on 256 and 320 rows);
    a last tile with fewer tokens than the table has rows, tokens that start on a multiple of four."""
    cfg = small("bf16", hidden=4 * d, num_heads=4, head_dim=d, rope="3d", rope_pairs=pairs, mlp_dim=256, num_layers=1)
    parity(cfg, [(1, 2, 2), (1, 20, 14), (2, 6, 10), (1, 12, 8)], gemm_tile=tile)
