"""GPU test that the tile a GEMM runs on does not show in the result: calls with few tokens, whose
GEMMs get 64-row tiles, give bit for bit what the 128 x 128 tile gives.  (Each output element is the
same chain of matrix instructions in every tile; rotary, row scales and the order in which the
sums of squares are added must not depend on the tile either.)"""

import pytest
import torch

from oracle import vit_encode as O
from paper_2601_11590_amd import binding as B, workloads as W
from parity_util import check
from test_gpu_parity import case, small

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kw, grids", [
    (dict(hidden=1024, num_heads=16, mlp_dim=4096, num_layers=2), [(1, 28, 28)]),       # 16 sums of 64 columns: the held loads
    (dict(hidden=1024, num_heads=16, mlp_dim=8192, num_layers=1), [(1, 26, 40)]),       # the same 16 sums in a 256 x 256 tile (first MLP GEMM)
    (dict(hidden=512, num_heads=8, mlp_dim=1024), [(1, 14, 18), (1, 2, 2)]),            # 8 sums of 64 columns
    (dict(hidden=384, num_heads=6, mlp_dim=1088), [(1, 14, 18), (1, 12, 10)]),          # the summing loop
    (dict(hidden=2048, num_heads=16, head_dim=128, rope_pairs=(0, 32, 32), mlp_dim=1024), [(1, 16, 20)]),
    (dict(hidden=144, num_heads=2, head_dim=72, rope_pairs=(0, 18, 18), norm="layernorm"), [(1, 14, 18), (1, 2, 6)]),
], ids=["d1024", "d1024-wide-mlp", "d512", "d384", "d2048", "d144-ln"])
def test_few_row_tiles_give_the_bits_of_the_128_tile(kw, grids):
    cfg = small("bf16", **kw)
    plan = B.epd_probe_gemm_plan(W.num_tokens(grids), cfg.hidden, cfg.hidden, B.EPI_RESIDUAL)
    assert plan[0] == 64, plan
    gw, layers, patches, cu, grid = case(cfg, grids)
    enc = B.EpdEncoder(cfg, gw, layers, max_tokens=patches.shape[0], max_segments=len(grids), max_items=len(grids))
    p = B.to_device_patches(patches, cfg.dtype)
    got = enc.encode(p, cu, grid).clone()
    enc.set_tuning(4, 0)
    want = enc.encode(p, cu, grid)
    torch.cuda.synchronize()
    assert torch.equal(got, want), "%d of %d values differ" % (int((got != want).sum()), got.numel())
    enc.close()


# K steps of 64 around the turns of a ring of three or four stages: 2 ... 7, and one (patch rows of 48 elements);
# merger pieces of whole steps and not (96, 72), Q | K columns that do not end on a 128-column boundary (96, 72)
@pytest.mark.parametrize("hidden,heads", [(128, 2), (192, 3), (256, 4), (320, 5), (384, 6), (448, 7), (96, 3), (72, 1)])
@pytest.mark.parametrize("act,norm", [("gelu_erf", "rmsnorm"), ("gelu_tanh", "layernorm")])
def test_forced_64_row_tiles_give_the_bits_of_the_128_tile(hidden, heads, act, norm):
    d = hidden // heads
    cfg = small("bf16", hidden=hidden, num_heads=heads, head_dim=d, rope_pairs=(0, d // 4, d // 2 - d // 4), mlp_dim=hidden + 72, act=act, norm=norm, out_dim=200)
    grids = [(1, 14, 18), (1, 2, 2), (1, 6, 10)]
    gw, layers, patches, cu, grid = case(cfg, grids)
    ref = O.encode(cfg, gw, layers, patches, cu, grid)
    enc = B.EpdEncoder(cfg, gw, layers, max_tokens=patches.shape[0], max_segments=len(grids), max_items=len(grids))
    p = B.to_device_patches(patches, cfg.dtype)
    out = {}
    for tile in (4, 7, 8):
        enc.set_tuning(tile, 0)
        out[tile] = enc.encode(p, cu, grid).clone()
    torch.cuda.synchronize()
    check(cfg, out[7].float().cpu().numpy(), ref, "64 x 64")
    assert torch.equal(out[7], out[4]) and torch.equal(out[8], out[4])
    enc.close()
