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


@pytest.mark.parametrize("patch,grid,size", [(4, (1, 10, 12), (61, 25)), (14, (1, 4, 6), (100, 151)), (16, (1, 6, 4), (7, 300))])
def test_interpolation_rounds_where_it_is_written_to(patch, grid, size):
    # fp32 outputs bit for bit: (1 - w) a + w b with w b rounded first, along the columns, then the rows, then
    # scale and shift.  Each step is a product of fp32 values (48 bits) plus an fp32 value, which
    # 64-bit significands hold; where an axis ends, its last pixel counts alone along the columns
    cfg = make("f32", patch=patch, tp=1)
    rng = np.random.default_rng(patch)
    px = rng.integers(0, 256, size=(3, 1) + size, dtype=np.uint8)
    gw, layers = W.all_weights(cfg)
    enc = B.EpdEncoder(cfg, gw, layers, max_tokens=W.num_tokens([grid]), max_segments=1, max_items=1)
    mean, std = np.float32([0.48, 0.46, 0.41]), np.float32([0.27, 0.26, 0.28])
    got = enc.preprocess(torch.from_numpy(px).reshape(-1).to("cuda:0"), [size], [grid], mean.tolist(), std.tolist()).cpu().numpy()
    enc.close()
    fma = lambda a, b, c: (a.astype(np.longdouble) * b + c).astype(np.float32)
    blend = lambda w, a, b: fma(np.float32(1) - w, a, w * b)

    def taps(n_in, n_out):
        num = np.maximum((2 * np.arange(n_out) + 1) * n_in - n_out, 0)
        i0 = np.minimum(num // (2 * n_out), n_in - 1)
        return i0, np.minimum(i0 + 1, n_in - 1), (num % (2 * n_out)).astype(np.float32) / np.float32(2 * n_out)

    x0, x1, wx = taps(size[1], grid[2] * patch)
    wx = np.where(x0 == x1, np.float32(1), wx)
    y0, y1, wy = taps(size[0], grid[1] * patch)
    f = px[:, 0].astype(np.float32)
    line = blend(wx[None, None, :], f[:, :, x0], f[:, :, x1])
    val = blend(wy[None, :, None], line[:, y0], line[:, y1])
    a = np.float32(1.0 / (255.0 * std.astype(np.float64)))
    b = np.float32(-mean.astype(np.float64) / std.astype(np.float64))
    want = fma(val, a[:, None, None], b[:, None, None])
    img = got.reshape(grid[1], grid[2], 3, patch, patch).transpose(2, 0, 3, 1, 4).reshape(want.shape)
    assert np.array_equal(img, want), "%d of %d differ" % ((img != want).sum(), img.size)
