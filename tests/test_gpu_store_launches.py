"""GPU tests of the store's kernels at the sizes where their launches change: the 16 KB groups and
the last words of the hash kernel (bit for bit against the oracle), and more items than one launch
of the copy kernel takes."""

import numpy as np
import pytest
import torch

from oracle import mm_store as S
from paper_2601_11590_amd import binding as B, workloads as W
from test_gpu_mm_store import MEAN, STD, make, pack, setup

pytestmark = pytest.mark.gpu
GROUP = 16384      # bytes a block of the hash kernel takes per group


@pytest.mark.parametrize("shift", [0, 1, 3])       # alignment of the first byte
def test_hash_at_the_edges_of_groups_and_words(shift):
    lens = [n for c in (1, 2, 3) for n in (c * GROUP - 5, c * GROUP - 4, c * GROUP - 3, c * GROUP, c * GROUP + 1, c * GROUP + 7)]
    rng = np.random.default_rng(shift)
    data = rng.integers(0, 256, size=shift + sum(lens), dtype=np.uint8)
    data[shift:shift + GROUP - 5] = 0               # zero words count, too
    data[shift + GROUP - 5:shift + 2 * GROUP] = 255
    store = B.MMStore(2 << 20)
    off = shift + np.concatenate([[0], np.cumsum(lens)])
    salts = [2 ** 64 - 1 - i for i in range(len(lens))]
    keys = store.hash(torch.from_numpy(data).to("cuda:0"), off, salts)
    for i, n in enumerate(lens):
        assert (int(keys[i, 0]), int(keys[i, 1])) == S.hash128(data[off[i]:off[i + 1]].tobytes(), salts[i]), n
    store.close()


@pytest.mark.parametrize("dtype,out_dim", [("bf16", 8), ("f32", 3)])     # rows of 16 and of 12 bytes
def test_more_cached_items_than_one_copy_launch_takes(dtype, out_dim):
    cfg = make(dtype, out_dim=out_dim)
    n = 70
    grids, src = [(1, 2, 2 + 2 * (i % 5)) for i in range(n)], [(8, 8 + i) for i in range(n)]
    items, enc, store, _ = setup(cfg, grids, src, 2 << 20)
    px = pack(items, range(n))
    out1, hit1, _ = enc.encode_cached(store, 3, px, src, grids, MEAN, STD)
    rows = enc.preprocess(px, src, grids, MEAN, STD)
    want = enc.encode(rows, *W.metadata(grids))
    out2, hit2, _ = enc.encode_cached(store, 3, px, src, grids, MEAN, STD)
    torch.cuda.synchronize()
    assert not hit1.any() and hit2.all()
    assert torch.equal(out1, want) and torch.equal(out2, want)
    store.close()
    enc.close()
