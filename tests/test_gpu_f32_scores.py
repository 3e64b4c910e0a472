"""GPU test of the fp32 attention where scores leave the range of fp32: keys whose score is -inf have weight
zero, also where they are all the keys of one wave's share."""

import numpy as np
import pytest

from oracle import vit_encode as O
from paper_2601_11590_amd import workloads as W
from parity_util import check, run_gpu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d,heads", [(64, 1), (72, 1), (8, 2), (128, 1)])
@pytest.mark.parametrize("first,last", [(32, 64), (40, 96), (64, 150)])
def test_keys_with_scores_of_minus_infinity_have_no_weight(d, heads, first, last):
    cfg = W.EncoderConfig(name="inf-scores", dtype="f32", num_layers=1, hidden=d * heads, num_heads=heads, head_dim=d, mlp_dim=64, patch=2,
                          temporal_patch=1, norm="rmsnorm", rope="none", rope_pairs=(0, 0, 0), out_dim=16, merge=1, seed=3)
    gw, layers = W.global_weights(cfg), [W.layer_weights(cfg, 0)]
    grids = [(1, 10, 15)]
    patches = W.packed_patches(cfg, grids)
    # the patch's first value, 0 or -1, becomes the token's first channel; the key's first channel is 1e25 times
    # it and the query's is 1e25, so a product is 0 or about -1e50
    patches[:, 0] = 0.0
    patches[first:last, 0] = -1.0
    gw["patch_w"][0], gw["patch_b"][0] = 0.0, 0.0
    gw["patch_w"][0, 0] = 1.0
    D, lw = cfg.hidden, layers[0]
    for h in range(heads):
        lw["qkv_w"][[h * d, D + h * d]] = 0.0
        lw["qkv_b"][[h * d, D + h * d]] = 1e25, 0.0
        lw["qkv_w"][D + h * d, 0] = 1e25
    cu, grid = W.metadata(grids)
    ref = O.encode(cfg, gw, layers, patches, cu, grid)
    assert np.isfinite(ref).all()
    check(cfg, run_gpu(cfg, gw, layers, patches, cu, grid), ref, "scores")
