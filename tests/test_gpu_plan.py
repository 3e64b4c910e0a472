"""GPU test of the call's metadata on both ways it travels -- kernel arguments up to 64 items and
segments, the pinned staging ring beyond -- and of segments that differ from the items."""

import numpy as np
import pytest

from oracle import vit_encode as O
from paper_2601_11590_amd import workloads as W
from parity_util import check, run_gpu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("n,segments", [(64, "item"), (65, "item"), (33, "frame")])
def test_plan_of_many_items(dtype, n, segments):
    cfg = W.EncoderConfig(name="plan-" + dtype, dtype=dtype, num_layers=1, hidden=128, num_heads=2, head_dim=64, mlp_dim=256, patch=4,
                          temporal_patch=1, norm="rmsnorm", rope="3d", rope_pairs=(8, 12, 12), out_dim=64, seed=11)
    rng = np.random.default_rng(n)
    grids = [(2 if segments == "frame" else int(rng.integers(1, 3)), 2 * int(rng.integers(1, 4)), 2 * int(rng.integers(1, 8))) for _ in range(n)]
    gw, layers = W.all_weights(cfg)
    patches = W.packed_patches(cfg, grids)
    cu, grid = W.metadata(grids, segments)
    check(cfg, run_gpu(cfg, gw, layers, patches, cu, grid), O.encode(cfg, gw, layers, patches, cu, grid), "%d items" % n)
