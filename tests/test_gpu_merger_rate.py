"""GPU test that gathering the merger's operand does not slow its GEMM down: the projection of 2 x 2 token windows
against the same M x N x K product of plain rows, both with the same tile forced and timed by the
library's own events.  The gathered one also reads the window list and cannot use the scalar row
addresses of plain rows: measured 1.05 (256 x 256), 1.24 (128 x 128) and 1.04 (320 x 256) times as long.  The large tiles run the
ping-pong loop on both; with the gathered one on the plain loop it was 1.22 and 1.20.  The 128 x 128 tile runs the plain
loop on both; with row numbers fetched between the loads of a stage, each waited for together with the loads
before it, it was 1.90.  The bounds stand between."""

import pytest
import torch

from paper_2601_11590_amd import binding as B, workloads as W
from test_gpu_parity import small

pytestmark = pytest.mark.gpu


def merge_step_us(cfg, grids, tile):
    gw, layers = W.all_weights(cfg)
    T = W.num_tokens(grids)
    enc = B.EpdEncoder(cfg, gw, layers, max_tokens=T, max_segments=len(grids), max_items=len(grids))
    enc.set_tuning(tile, 0)
    rows = torch.rand((T, cfg.patch_dim), device="cuda:0").to(torch.bfloat16)
    cu, grid = W.metadata(grids)
    times = []
    for _ in range(9):
        enc.set_timing(B.EPD_STEP_MERGE)
        for _ in range(4):
            enc.encode(rows, cu, grid)
        torch.cuda.synchronize()
        ms, launches = enc.get_timing()[:2]
        times.append(ms / launches * 1e3)
    enc.close()
    return sorted(times)[4]


@pytest.mark.parametrize("tile, most", [(0, 1.13), (4, 1.5), (5, 1.12)])
def test_gathered_merger_keeps_up_with_plain_rows(tile, most):
    base = dict(num_layers=0, mlp_dim=64, out_dim=4096)
    gathered = merge_step_us(small("bf16", hidden=1024, num_heads=16, merge=2, **base), [(1, 112, 224)], tile)
    plain = merge_step_us(small("bf16", hidden=4096, num_heads=64, merge=1, **base), [(1, 56, 112)], tile)
    print("tile %d: gathered %.1f us, plain rows %.1f us" % (tile, gathered, plain), flush=True)
    assert gathered <= most * plain, (gathered, plain)
