"""GPU parity of the 64-row bf16 GEMM tiles, which calls with few tokens get: against the oracle, at
token counts and widths on their edges.  Tolerances as for every bf16 case (per-token cosine >= 0.999,
max-norm relative error <= 2e-2)."""

import pytest

from paper_2601_11590_amd import workloads as W
from test_gpu_parity import parity, small

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kw, grids, residual_tile", [
    # 4 rows; one K step (patch row of 48); sums of squares of 4 segments
    (dict(), [(1, 2, 2)], (64, 64)),
    # 64 + 1 token-tile edges, K of 5 steps (odd), segments neither 8 nor 16: the summing loop
    (dict(hidden=320, num_heads=5, mlp_dim=1088, out_dim=328), [(1, 8, 8), (1, 2, 2)], (64, 64)),
    (dict(hidden=384, num_heads=6, mlp_dim=1088), [(1, 16, 10), (1, 14, 18), (1, 2, 2)], (64, 64)),
    # hidden 1024: sixteen 64-column sums held in registers; 64 x 64 tiles for N = 1024
    (dict(hidden=1024, num_heads=16, mlp_dim=1024, num_layers=2), [(1, 14, 18), (1, 12, 14), (1, 2, 38)], (64, 64)),
    # enough rows for 64 x 128 tiles on the residual GEMMs (128-column sums)
    (dict(hidden=1024, num_heads=16, mlp_dim=1024, num_layers=2), [(1, 30, 38), (1, 34, 38), (1, 2, 2)], (64, 128)),
    # merger pieces that are not whole K steps (216), ragged K, LayerNorm
    (dict(hidden=216, num_heads=3, head_dim=72, rope_pairs=(0, 18, 18), norm="layernorm", mlp_dim=520), [(1, 6, 10), (2, 4, 4)], (64, 64)),
], ids=["4-rows", "d320", "d384", "d1024", "d1024-wide", "d216"])
def test_few_rows(kw, grids, residual_tile):
    from paper_2601_11590_amd import binding as B
    cfg = small("bf16", **kw)
    plan = B.epd_probe_gemm_plan(W.num_tokens(grids), cfg.hidden, cfg.hidden, B.EPI_RESIDUAL)
    assert tuple(plan[:2]) == residual_tile and plan[2] == 0, plan
    parity(cfg, grids)


def test_one_image_of_the_chat_encoder_two_layers():
    parity(W.C2.replace(num_layers=2), [(1, 28, 28)])
