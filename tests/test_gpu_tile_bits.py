"""GPU test that the tile a GEMM runs on does not show in the result: calls with few tokens, whose
GEMMs get 64-row tiles, give bit for bit what the 128 x 128 tile gives.  (Each output element is the
same chain of matrix instructions in every tile; rotary, row scales and the order in which the
sums of squares are added must not depend on the tile either.)"""

import pytest
import torch

from paper_2601_11590_amd import binding as B, workloads as W
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
