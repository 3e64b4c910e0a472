"""GPU tests of the preprocessing kernel at the sizes where its index arithmetic can go wrong: blocks
of several tokens that end inside a row or a slice, the smallest and largest patch, sources of one or
two pixels, strong up- and downscaling; and of the weights it interpolates with, exactly."""

import numpy as np
import pytest
import torch

from paper_2601_11590_amd import binding as B, workloads as W
from test_gpu_preprocess import compare, make, run

pytestmark = pytest.mark.gpu

CASES = {
    "patch2-two-frames": (2, 2, [(1, 2, 130), (1, 34, 6), (1, 2, 2)], [(4, 260), (31, 77), (9, 1)]),
    "patch14-two-frames": (14, 2, [(3, 2, 4), (2, 4, 6), (1, 2, 2)], [(28, 56), (1, 1), (200, 2)]),
    "patch16": (16, 1, [(1, 2, 6), (1, 6, 2), (1, 4, 4)], [(1, 97), (333, 1), (64, 65)]),
    "patch32-five-frames": (32, 5, [(1, 2, 2), (2, 2, 4)], [(64, 64), (300, 3)]),
}


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("name", CASES)
def test_preprocess_at_odd_sizes(name, dtype):
    patch, tp, grids, src = CASES[name]
    cfg = make(dtype, patch=patch, tp=tp)
    enc, got, ref, _ = run(cfg, grids, src)
    compare(cfg, got, ref)              # the bounds of test_gpu_preprocess.py: fp32 1e-5, bf16 one unit in the last place
    enc.close()


@pytest.mark.parametrize("axis", ["columns", "rows"])
@pytest.mark.parametrize("n_in,patches,patch", [(37, 50, 4), (301, 50, 4), (499, 32, 14), (1920, 32, 14), (3, 64, 2), (16383, 28, 16)])
def test_tap_weights_are_the_correctly_rounded_quotients(axis, n_in, patches, patch):
    # pixels 0, 1, 0, 1 ... along one axis, equal along the other, mean 0: an fp32 output between a 0 and a 1
    # is the second tap's weight times the scale, rounded, one between a 1 and a 0 the same of 1 - weight,
    # and the weight is r / (2 n_out) rounded once
    std = np.float32(1.0 / 255.0)
    scale = np.float32(1.0 / (255.0 * float(std)))
    cfg = make("f32", patch=patch, tp=1)
    n_out = patches * patch
    line = (np.arange(n_in) & 1).astype(np.uint8)
    flat = 2 * patch                                     # the other axis: two patches, not resized
    grid, size = ((1, 2, patches), (flat, n_in)) if axis == "columns" else ((1, patches, 2), (n_in, flat))
    frame = np.broadcast_to(line[None, :] if axis == "columns" else line[:, None], size)
    px = torch.from_numpy(np.ascontiguousarray(np.broadcast_to(frame, (3, 1) + size))).reshape(-1).to("cuda:0")
    gw, layers = W.all_weights(cfg)
    enc = B.EpdEncoder(cfg, gw, layers, max_tokens=2 * patches, max_segments=1, max_items=1)
    got = enc.preprocess(px, [size], [grid], [0.0] * 3, [float(std)] * 3).cpu().numpy()
    enc.close()
    # back to an image: rows of (channel, row in patch, column in patch)
    img = got.reshape(grid[1], grid[2], 3, patch, patch).transpose(2, 0, 3, 1, 4).reshape(3, grid[1] * patch, grid[2] * patch)
    num = np.maximum((2 * np.arange(n_out) + 1) * n_in - n_out, 0)
    q, r = num // (2 * n_out), num % (2 * n_out)
    w = r.astype(np.float32) / np.float32(2 * n_out)
    lo, hi = line[np.minimum(q, n_in - 1)], line[np.minimum(q + 1, n_in - 1)]
    want = np.where(lo == hi, lo.astype(np.float32), np.where(hi == 1, w, np.float32(1) - w))
    want = (want.astype(np.float64) * float(scale)).astype(np.float32)
    want = np.broadcast_to(want[None, None, :] if axis == "columns" else want[None, :, None], img.shape)
    assert np.array_equal(img, want), "%d of %d differ" % ((img != want).sum(), img.size)
