"""GPU tests of the preprocessing kernel at the sizes where its index arithmetic can go wrong: blocks
of several tokens that end inside a row or a slice, the smallest and largest patch, sources of one or
two pixels, strong up- and downscaling."""

import pytest

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
